"""Full-covariance sampling with a factor whose entries are not finite in single precision: an infinite sum saturates at
the velocity bound by its sign, a sum that is not a number at the lower bound, and every other row keeps its bits.
Reference: the IEEE product of the same normals with the factor in single precision."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

BIG = float(np.finfo(np.float32).max)


@pytest.mark.parametrize("K,H", [(1, 1), (33, 3), (100, 20)])
def test_a_factor_with_entries_that_are_not_finite(K, H):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    scene = mp.Scene(ctx, W.make_scene(1))
    n, u = 14 * H, 0.9
    rng = np.random.default_rng(K + H)
    nu = rng.normal(0, 0.1, (H, 14)).astype(np.float32)
    L = np.tril(rng.normal(0, 0.3, (n, n)) / np.sqrt(n)) + 0.2 * np.eye(n)
    plain = L.copy()
    rows = {1: [(0, np.inf)], 3: [(3, -np.inf)], 4: [(1, np.nan)], 6: [(2, np.inf), (5, -np.inf)], 7: [(7, np.inf), (0, np.inf)],
            8: [(4, BIG)], 9: [(9, -BIG)], 10: [(0, 1e300)], 11: [(11, -1e300)], n - 1: [(n // 2, np.inf)]}
    for i, e in rows.items():
        for p, v in e:
            L[i, p] = v
    z = np.zeros((K, H, 14), np.float32)
    mp.mppi_sample(ctx, scene, nu, np.full(14, 0.3, np.float32), 5, 2, K, z=z)
    z = z.reshape(K, n).astype(np.float64)
    out = {}
    for name, f in (("plain", plain), ("given", L)):
        U = np.zeros((K, H, 14), np.float32)
        mp.mppi_sample_full(ctx, nu, f + np.triu(np.full((n, n), np.inf), 1), 5, 2, K, U, u)
        out[name] = U.reshape(K, n)
    rest = [i for i in range(n) if i not in rows]
    assert np.array_equal(out["given"][:, rest], out["plain"][:, rest])
    with np.errstate(over="ignore", invalid="ignore"):
        L32 = L.astype(np.float32).astype(np.float64)
        for i in rows:
            s = nu.reshape(n)[i] + (z[:, :i + 1] * L32[i, :i + 1]).sum(1)
            want = np.where(np.isnan(s), -u, np.clip(s, -u, u)).astype(np.float32)
            assert np.array_equal(out["given"][:, i], want), (i, out["given"][:, i][:8], want[:8])
    ctx.close()
