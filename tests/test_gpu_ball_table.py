"""The ball's contact with the table alone, which the kernels solve by a path of its own (its sweep skips the
narrowphase dispatch, its solve the products by the normal's zeros): one substep against the FP64 oracle over depths,
velocities, spins, friction and sweep counts, without boxes and with the most boxes a scene holds (three blocks of
candidate pairs).  Tolerance: 1e-5 of each state group's largest magnitude, the one-substep parity bound."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mapping", ["lane", "team", "wave", "split"])
@pytest.mark.parametrize("boxes,mu,n_pgs,n_cmax", [(0, 1.0, 20, 4), (3, 0.3, 20, 4), (16, 1.7, 1, 4), (3, 1.0, 20, 1),
                                                   (3, 1.0, 20, 0)])
def test_one_substep_with_the_ball_on_the_table(oracle_mod, mapping, boxes, mu, n_pgs, n_cmax):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    sc = W.make_scene(2, n_box=boxes, mu=mu, n_pgs=n_pgs, n_cmax=n_cmax)
    scene, o = mp.Scene(ctx, sc), oracle_mod.Oracle(sc)
    n = 70
    rng = np.random.default_rng(17)
    X = np.tile(W.initial_state(sc), (n, 1))
    X[:, 14:28] = rng.uniform(-0.3, 0.3, (n, 14))
    X[:, 44] = sc["ball_r"] - rng.uniform(-0.0005, 0.004, n)  # a few stay above the table
    X[:, 49:52] = rng.uniform(-1.0, 1.0, (n, 3))
    X[:, 52:55] = rng.uniform(-5.0, 5.0, (n, 3))
    X = X.astype(np.float32)
    U = rng.uniform(-1.0, 1.0, (n, 1, 14)).astype(np.float32)
    out = torch.zeros((n, 55), device="cuda")
    mp.mppi_simulate(ctx, scene, torch.tensor(X, device="cuda"), torch.tensor(U, device="cuda"), X_out=out, n_sub=1,
                     mapping=mapping)
    got = out.cpu().numpy().astype(np.float64)
    ones = 0
    for i in range(n):
        want, nc = o.substep(X[i].astype(np.float64), U[i, 0].astype(np.float64))
        ones += nc == 1
        for a, b in ((0, 14), (14, 28), (28, 42), (42, 45), (45, 49), (49, 52), (52, 55)):
            scale = max(np.abs(want[a:b]).max(), 1e-3)
            assert np.abs(got[i, a:b] - want[a:b]).max() <= 1e-5 * scale, (i, a, nc)
    assert n > ones > n // 2 if n_cmax else ones == 0
    ctx.close()


@pytest.mark.parametrize("boxes,spread", [(0, 0.9), (3, 0.6), (16, 0.6), (16, 0.05)])
def test_coarse_test_of_the_team_form_misses_no_pair(boxes, spread):
    """The four-samples-a-wave form skips its sweeps when joined boxes rule every pair out; one sample a wave always
    sweeps.  Random arm poses (arms against boxes, table, ball and each other, some states far from everything)
    give the same bits in both, states, costs and every cost term."""
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    sc = W.make_scene(3, n_box=boxes)
    scene = mp.Scene(ctx, sc)
    n, H = 253, 3
    X = torch.tensor(W.random_states(sc, n, seed=9, spread=spread).astype(np.float32), device="cuda")
    U = torch.tensor(W.random_controls(n, H, 4).astype(np.float32), device="cuda")
    got = {}
    for m in ("team", "wave", "split"):
        got[m] = [torch.zeros(s, device="cuda") for s in ((n,), (n, mp.NTERMS), (n, 55))]
        mp.mppi_simulate(ctx, scene, X, U, got[m][0], got[m][1], got[m][2], mapping=m)
    for m in ("wave", "split"):
        for a, b in zip(got["team"], got[m]):
            assert torch.equal(a, b)
    if spread > 0.5 and boxes:  # the poses do reach the boxes
        assert (got["team"][1][:, 5] > 0).sum() >= boxes // 2
    ctx.close()
