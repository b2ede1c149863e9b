"""Full-covariance sampling at the edges of its tiles (16 x 32 operand blocks, 32 x 64 output tiles): sample counts and
horizons around them, an odd number of sample blocks, against the FP64 product of the same normals.  Tolerance: the
FP32 accumulation of at most n terms of size |L z|, 5e-5 as for the other sizes."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,H", [(1, 1), (15, 2), (16, 3), (17, 5), (31, 7), (32, 8), (33, 9), (48, 16), (63, 17), (65, 23),
                                 (129, 32)])
def test_sample_full_at_tile_edges(K, H):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    scene = mp.Scene(ctx, W.make_scene(1))
    n = 14 * H
    rng = np.random.default_rng(100 * K + H)
    nu = rng.normal(0, 0.1, (H, 14)).astype(np.float32)
    A = rng.normal(0, 0.3, (n, n)) / np.sqrt(n)
    L = np.tril(A) + 0.2 * np.eye(n)
    Lfull = L + np.triu(np.full((n, n), np.nan), 1)  # the upper triangle is not read
    z = np.zeros((K, H, 14), np.float32)
    mp.mppi_sample(ctx, scene, nu, np.full(14, 0.3, np.float32), 5, 2, K, z=z)
    U = np.zeros((K, H, 14), np.float32)
    mp.mppi_sample_full(ctx, nu, Lfull, 5, 2, K, U, 0.9)
    ref = np.clip(nu.astype(np.float64).reshape(1, n) + z.astype(np.float64).reshape(K, n) @ L.T, -0.9, 0.9)
    assert np.abs(U.reshape(K, n) - ref).max() < 5e-5
    ctx.close()
