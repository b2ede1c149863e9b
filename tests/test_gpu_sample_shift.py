"""Full-covariance sampling has no common shift: the mean error of all entries against the FP64 product of the same
normals.  Bound: 1e-8 of their standard deviation, a sixth of single precision's unit roundoff (independent roundings
of 3e-7 over the 900000 entries would leave 3e-10)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_mean_error():
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    scene = mp.Scene(ctx, W.make_scene(1))
    K, H = 1024, 64
    n = 14 * H
    rng = np.random.default_rng(11)
    A = rng.normal(0, 0.3, (64, n))
    L = torch.tensor(np.linalg.cholesky(0.045 * np.eye(n) + 0.5 / 64 * A.T @ A), device="cuda")
    nu = torch.zeros((H, 14), device="cuda")
    z, U = torch.zeros((K, H, 14), device="cuda"), torch.zeros((K, H, 14), device="cuda")
    mp.mppi_sample(ctx, scene, nu, torch.full((14,), 0.3, device="cuda"), 5, 0, K, z=z)
    mp.mppi_sample_full(ctx, nu, L.contiguous(), 5, 0, K, U, 100.0)
    ref = z.double().reshape(K, n) @ L.T.contiguous()
    assert abs((U.double().reshape(K, n) - ref).mean()) < 1e-8 * ref.std()
    ctx.close()
