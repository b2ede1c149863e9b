"""The two forms of the QP smoothing, between which the sample count chooses: within a form a sequence's bits do not
depend on what it is projected with; across the line they differ by rounding.  Tolerance with the default bounds: each
form is held to 2e-5 rad/s of the FP64 iteration, so the two to twice that."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,line", [(17, 256), (32, 256), (33, 512), (64, 512), (100, 512), (128, 512)])
def test_the_forms_agree_across_the_line(H, line):
    import paper_2511_21264_amd as mp
    ctx, sc, p = mp.Context(0), W.make_scene(2), W.qp_params(2)
    scene = mp.Scene(ctx, sc)
    rng = np.random.default_rng(H)
    U = (rng.normal(0, 0.3, (line + 41, H, 14)) + 0.3 * np.sin(np.arange(H) * 0.2)[None, :, None]).astype(np.float32)
    x0 = torch.tensor(W.initial_state(sc).astype(np.float32), device="cuda")

    def project(a, b):
        out = torch.tensor(U[a:b], device="cuda")
        mp.mppi_project(ctx, scene, x0, out, out, p, x0_shared=True)
        return out.cpu().numpy()

    few, part, many, more = project(0, line), project(3, 40), project(0, line + 1), project(0, line + 41)
    assert np.array_equal(few[3:40], part) and np.array_equal(many, more[:line + 1])
    assert 0.0 < np.abs(few - many[:line]).max() <= 4e-5
    ctx.close()
