"""The coarse test of the team, wave and split forms (joined boxes that rule the pair sweeps out) where one pair alone
is near: states in which a single candidate pair other than the ball on the table touches, or a single cost pair lies
within the cost margin, so that nothing else can send the kernel into its sweep.  Every state fills a wave of four
teams.  References: the forms for further cost terms (weights zero), which always sweep, bit for bit with their work
counters; the FP64 oracle for the pair itself, one substep to ten times the one-substep parity bound (1e-5 of each
state group's largest magnitude; picked for grazing contact, not for well-conditioned ones) and the terms of two control
steps to 1e-4 of the largest."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

GROUPS = ((0, 14), (14, 28), (28, 42), (42, 45), (45, 49), (49, 52), (52, 55))


def _scene(name):
    sc = W.make_scene(3, n_box=16 if name == "boxes" else 0, n_sub=1)
    if name == "close":  # arms that reach each other
        sc["base_pos"] = np.asarray(sc["base_pos"], dtype=np.float64) * [0.7, 1.0, 1.0]
    return sc


def _kind(a, b):
    what = lambda g: "ball" if g == 0 else "table" if g == 1 else "box" if g >= 16 else "arm"  # noqa: E731
    return what(a) + "-" + what(b)


def _single_pair_states(o, sc, name):
    """{kind: states} with one touching pair, {kind + " margin": states} with one pair within the cost margin."""
    n, each = 6000, 6
    X = W.random_states(sc, n, seed=3, spread=0.3 if name == "ball" else 0.9)
    rng = np.random.default_rng(4)
    up = rng.random(n) < (0.0 if name == "ball" else 0.6 if name == "boxes" else 1.0)
    far = [[-0.5, -0.6, 0.1], [0.5, 0.6, 0.8]] if name == "boxes" else [[2.0, 2.0, 2.0], [3.0, 3.0, 3.0]]
    X[up, 42:45] = rng.uniform(far[0], far[1], (int(up.sum()), 3))
    X = X.astype(np.float32)
    ga, gb = o.pairs()
    kinds = np.array([_kind(a, b) for a, b in zip(ga, gb)])
    table, cost = kinds == "ball-table", (kinds == "arm-arm") | (kinds == "arm-box")
    found = {}
    for x in X:
        lo, hi = o.aabbs(x.astype(np.float64))
        near = o.broadphase(lo, hi).astype(bool) & ~table
        close = o.broadphase(lo, hi, sc["m_c"]).astype(bool) & cost
        if near.sum() + close.sum() == 0 or near.sum() > 1 or (near.sum() == 0 and close.sum() > 1):
            continue
        phi = o.narrow_all(x.astype(np.float64))[0]
        if near.sum() == 1 and phi[near][0] < -1e-4:
            found.setdefault(kinds[near][0], []).append(x)
        if near.sum() == 0 and phi[close][0] < sc["m_c"] - 1e-3:
            found.setdefault(kinds[close][0] + " margin", []).append(x)
    return {k: np.stack(v[:each]) for k, v in found.items()}


WANTED = {"boxes": {"arm-table", "ball-box", "arm-box", "arm-box margin"}, "ball": {"arm-table", "ball-arm"},
          "close": {"arm-arm", "arm-arm margin"}}


@pytest.mark.parametrize("name", sorted(WANTED))
def test_no_single_pair_is_missed(oracle_mod, name):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    sc = _scene(name)
    o = oracle_mod.Oracle(sc)
    states = _single_pair_states(o, sc, name)
    assert WANTED[name] <= set(states), {k: len(v) for k, v in states.items()}
    scene, ext = mp.Scene(ctx, sc), mp.Scene(ctx, dict(sc, ext=1))
    forms = [("team", scene), ("wave", scene), ("split", scene), ("wave", ext), ("split", ext)]
    X = np.concatenate([states[k] for k in sorted(states)])
    X = np.repeat(X, 4, axis=0)  # a state fills a wave of four teams
    n, H = len(X), 2
    U = np.repeat(np.random.default_rng(6).uniform(-0.5, 0.5, (n // 4, H, 14)), 4, axis=0).astype(np.float32)
    dX, dU = torch.tensor(X, device="cuda"), torch.tensor(U, device="cuda")
    got = {}
    for m, s in forms:
        r = [torch.zeros(d, device="cuda") for d in ((n,), (n, mp.NTERMS), (n, 55))]
        one = torch.zeros((n, 55), device="cuda")
        mp.mppi_simulate(ctx, s, dX, dU, *r, mapping=m)
        mp.mppi_simulate(ctx, s, dX, dU[:, :1].contiguous(), X_out=one, mapping=m)
        got[m, s is ext] = [r[0].cpu(), r[1][:, :7].cpu(), r[2].cpu(), one.cpu()]
    for f in got:
        for a, b in zip(got["wave", True], got[f]):
            assert torch.equal(a, b), (f, [int(i) // 4 for i in (a != b).reshape(n, -1).any(1).nonzero()[::4, 0]])
    terms, one = got["wave", True][1].numpy(), got["wave", True][3].numpy().astype(np.float64)
    for i in range(0, n, 4):
        x = X[i].astype(np.float64)
        want, nc = o.substep(x, U[i, 0].astype(np.float64))
        for a, b in GROUPS:
            scale = max(np.abs(want[a:b]).max(), 1e-3)
            assert np.abs(one[i, a:b] - want[a:b]).max() <= 1e-4 * scale, (i, a, nc)
        t = o.rollout(x, U[i].astype(np.float64))[1]
        assert np.abs(terms[i] - t[:7]).max() <= 1e-4 * max(np.abs(t[:7]).max(), 1.0), (i, terms[i], t[:7])
    # the work counters of one control step: every pair that the sweep tests, none beside
    sig, nom = np.full(14, 0.3, np.float32), np.zeros((1, 14), np.float32)
    for x in np.ascontiguousarray(X[::4]):
        st = []
        for m, s in forms:
            U_new = np.zeros((1, 14), np.float32)
            r = mp.mppi_plan(ctx, s, x.copy(), nom, 4, 1, 0.1, sig, U_new, np.zeros(4, np.float32), M=1, seed=1, mapping=m)
            st.append([r[k] for k in ("contacts", "np_tests", "box_tests", "overflow")])
        assert all(v == st[0] for v in st[1:]), st
    ctx.close()
