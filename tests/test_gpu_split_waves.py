"""The two waves of the split form, of which one owns the arms and one the ball: rollouts that go in and out of arm
contact, through boxes and past them, with and without room in the contact list, against the sixteen-lane form bit for
bit (states, costs, every term), and against the forms with further cost terms (of weight zero), which always sweep
(up to four contacts: beyond, those forms' solves sum in another order)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boxes,spread,n_cmax", [(0, 0.9, 4), (0, 0.9, 8), (3, 0.6, 4), (16, 0.6, 4), (16, 0.6, 8),
                                                 (8, 0.3, 1), (3, 0.6, 0)])
def test_split_form_equals_the_others(boxes, spread, n_cmax):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    sc = W.make_scene(5, n_box=boxes, n_cmax=n_cmax)
    scene = mp.Scene(ctx, sc)
    n, H = 130, 6
    X = W.random_states(sc, n, seed=13, spread=spread)
    X[::2, 42:45] = [0.0, 0.0, sc["ball_r"] - 0.001]  # every other ball rests on the table
    X = torch.tensor(X.astype(np.float32), device="cuda")
    U = torch.tensor(W.random_controls(n, H, 6).astype(np.float32), device="cuda")
    got = {}
    ext = mp.Scene(ctx, dict(sc, ext=1))
    for m, s in (("team", scene), ("wave", scene), ("split", scene), ("wave", ext), ("split", ext)):
        if s is ext and n_cmax > 4:
            continue
        r = [torch.zeros(d, device="cuda") for d in ((n,), (n, mp.NTERMS), (n, 55))]
        mp.mppi_simulate(ctx, s, X, U, *r, mapping=m)
        got[m, s is ext] = r[0], r[1][:, :7], r[2]
    for m in got:
        for a, b in zip(got["team", False], got[m]):
            assert torch.equal(a, b), m
    ctx.close()
