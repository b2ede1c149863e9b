"""The QP smoothing's tile form where position bounds hold over much of the horizon: the right-hand side of its product
then grows to hundreds of units that the matrix all but cancels.  Its error against the FP64 iteration, of the result's
norm, must be no larger than that of the other form (taken for few samples) on the same sequences: an order between the
two, without a tolerance."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,few,many", [(17, 256, 257), (32, 256, 270), (33, 512, 513), (48, 512, 520), (64, 512, 515),
                                        (80, 512, 516), (100, 512, 517), (112, 512, 513), (128, 512, 514)])
@pytest.mark.parametrize("room,rho,iters", [(1.5, 3.0, 1), (1.5, 3.0, 60), (0.05, 3.0, 60), (0.05, 1.0, 60), (0.05, 10.0, 60),
                                            (0.01, 3.0, 60), (0.05, 3.0, 200)])
def test_tile_form_is_no_less_exact(H, few, many, room, rho, iters):
    import paper_2511_21264_amd as mp
    from oracle import qp as qpo
    ctx, sc = mp.Context(0), W.make_scene(2)
    scene = mp.Scene(ctx, sc)
    x0 = W.initial_state(sc).astype(np.float32)
    p = W.qp_params(2, iters=iters, rho=rho, pos_lo=x0[28:42] - room, pos_hi=x0[28:42] + room)
    rng = np.random.default_rng(H)
    U = (rng.normal(0, 0.3, (many, H, 14)) + 0.3 * np.sin(np.arange(H) * 0.2)[None, :, None]).astype(np.float32)
    n = 12
    ref = qpo.project_sequences(U[:n].astype(np.float64), np.tile(x0[28:42].astype(np.float64), (n, 1)),
                                sc["h"] * sc["n_sub"], float(sc["u_max"]), np.float32(p["pos_lo"]).astype(np.float64),
                                np.float32(p["pos_hi"]).astype(np.float64), p["acc_max"], p["jerk_max"], p["rho"],
                                p["iters"], p["alpha"])
    err = []
    for K in (few, many):
        out = torch.tensor(U[:K], device="cuda")
        mp.mppi_project(ctx, scene, torch.tensor(x0, device="cuda"), out, out, p, x0_shared=True)
        err.append(np.linalg.norm(out[:n].cpu().numpy() - ref) / np.linalg.norm(ref))
    ctx.close()
    assert err[1] <= err[0], err
