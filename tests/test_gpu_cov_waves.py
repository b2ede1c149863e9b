"""Covariance update at the edges of its launch rule (eight waves a tile past 128 samples and up to 256 tiles, else
four; groups of four samples, steps of eight groups a wave), with weightless samples that hold NaN, against the FP64
oracle.  Tolerance: FP64 sums in another order, 1e-12 of the largest entry as for the other sizes."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# n = 14 H: H = 50 is 253 tiles, H = 51 is 276
@pytest.mark.parametrize("K,H", [(128, 3), (129, 3), (131, 1), (255, 7), (257, 9), (513, 2), (200, 50), (200, 51)])
def test_cov_update_at_wave_edges(K, H):
    import paper_2511_21264_amd as mp
    from oracle import cov
    rng = np.random.default_rng(1000 * K + H)
    n = 14 * H
    nu = rng.normal(0, 0.1, n)
    U = (nu + rng.normal(0, 0.3, (K, n))).astype(np.float32)
    w = rng.random(K)
    w[::3] = 0.0
    w /= w.sum()
    A = rng.normal(0, 0.3, (n, n)) / np.sqrt(n)
    S = 0.09 * (A @ A.T + 0.1 * np.eye(n))
    ref = cov.cov_update(U.astype(np.float64), w, nu, S, 0.4, 1e-4)
    U[::3] = np.nan  # contributes nothing
    ctx = mp.Context(0)
    out = torch.zeros((n, n), dtype=torch.float64, device="cuda:0")
    mp.mppi_cov_update(ctx, *(torch.tensor(a, device="cuda:0") for a in (U, w, nu, S)), out, 0.4, 1e-4)
    got = out.cpu().numpy()
    ctx.close()
    assert np.abs(got - ref).max() < 1e-12 * np.abs(ref).max()
