"""The QP smoothing's tile form (one wave per sixteen joint sequences; taken from 257 samples on up to H = 32, from
513 on beyond) against the FP64 oracle's ADMM: every number of 16-step blocks, horizons at and around their edges,
sample counts that leave the last tile ragged, and the samples drawn in the kernel (mppi_plan_qp).  Tolerance as for
the other form (2e-5 rad/s; its error over the whole iteration is no larger)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def T(a):
    return torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("K,H", [(257, 17), (259, 31), (300, 32), (513, 33), (515, 48), (520, 63), (513, 64), (517, 65),
                                 (514, 80), (513, 96), (516, 100), (519, 112), (513, 127), (521, 128)])
def test_tile_form_matches_oracle(K, H):
    import paper_2511_21264_amd as mp
    from oracle import qp as qpo
    ctx, sc, p = mp.Context(0), W.make_scene(2), W.qp_params(2)
    scene = mp.Scene(ctx, sc)
    rng = np.random.default_rng(1000 * H + K)
    U = (rng.normal(0, 0.3, (K, H, 14)) + 0.3 * np.sin(np.arange(H) * 0.2)[None, :, None]).astype(np.float32)
    X0 = np.repeat(W.initial_state(sc)[None], K, axis=0)
    X0[:, 28:42] += rng.uniform(-1.4, 1.4, (K, 14))
    X0 = X0.astype(np.float32)
    out = T(U)
    mp.mppi_project(ctx, scene, T(X0), out, out, p)  # in place
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    rows = np.r_[0:6, K // 2:K // 2 + 3, K - 6:K]
    ref = qpo.project_sequences(U[rows].astype(np.float64), X0[rows, 28:42].astype(np.float64), sc["h"] * sc["n_sub"],
                                float(sc["u_max"]), np.float32(p["pos_lo"]).astype(np.float64),
                                np.float32(p["pos_hi"]).astype(np.float64), p["acc_max"], p["jerk_max"], p["rho"],
                                p["iters"], p["alpha"])
    assert np.abs(out[rows] - ref).max() < 2e-5
    assert np.abs(out).max() <= np.float32(sc["u_max"]) and (out != U).any(axis=(1, 2)).all()
    ctx.close()


def test_tile_form_draws_the_plan_samples():
    """One plan iteration with the projection in the kernel equals its stages: sampled normals, projected, rolled out."""
    import paper_2511_21264_amd as mp
    ctx, sc, p = mp.Context(0), W.make_scene(2), W.qp_params(2)
    scene = mp.Scene(ctx, sc)
    K, H = 300, 20
    x0, nom, sig = T(W.initial_state(sc)), T(np.zeros((H, 14))), T(np.full(14, 0.3))
    U_new, costs = torch.zeros((H, 14), device="cuda"), torch.zeros(K, device="cuda")
    mp.mppi_plan_qp(ctx, scene, x0, nom, K, H, 0.1, sig, p, U_new, costs, M=1, seed=7, mapping="split")
    z = torch.zeros((K, H, 14), device="cuda")
    mp.mppi_sample(ctx, scene, nom, sig, 7, 0, K, z=z)
    U = (sig * z).contiguous()
    mp.mppi_project(ctx, scene, x0, U, U, p, x0_shared=True)
    again = torch.zeros(K, device="cuda")
    mp.mppi_simulate(ctx, scene, x0, U, again, x0_shared=True, mapping="split")
    torch.cuda.synchronize()
    assert torch.equal(costs, again)
    ctx.close()
