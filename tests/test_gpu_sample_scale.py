"""Full-covariance sampling over the scales of single precision: a factor and a mean scaled by a power of two scale the
samples, so the error against the FP64 product stays what it is at scale one.  Tolerance: the FP32 accumulation of the
sampling tests, 5e-5 of the scale, over 100 (no term is near the largest sum there)."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [-117, -100, -40, 0, 40, 90, 100])
def test_error_does_not_depend_on_the_scale(power):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    scene = mp.Scene(ctx, W.make_scene(1))
    K, H = 50, 9
    n, scale = 14 * H, 2.0 ** power
    rng = np.random.default_rng(3)
    nu = (rng.normal(0, 0.1, (H, 14)) * scale).astype(np.float32)
    L = (np.tril(rng.normal(0, 0.3, (n, n)) / np.sqrt(n)) + 0.2 * np.eye(n)) * scale
    z = np.zeros((K, H, 14), np.float32)
    mp.mppi_sample(ctx, scene, nu, np.full(14, 0.3, np.float32), 5, 0, K, z=z)
    U = np.zeros((K, H, 14), np.float32)
    mp.mppi_sample_full(ctx, nu, L, 5, 0, K, U, float(100 * scale))
    ref = nu.astype(np.float64).reshape(1, n) + z.astype(np.float64).reshape(K, n) @ L.T
    assert np.abs(U.reshape(K, n) - ref).max() < 5e-7 * scale
    ctx.close()
