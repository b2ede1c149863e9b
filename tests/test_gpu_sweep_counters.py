"""The work counters (contacts, narrowphase and box tests, full lists) of the forms that may skip or shorten the pair
sweep, against the forms for further cost terms (weights zero), which always run it: for every capacity of the contact
list, none included, with the ball alone on the table and with arms among boxes."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_cmax", [0, 1, 2, 4])
@pytest.mark.parametrize("boxes,spread", [(0, 0.0), (3, 0.6), (16, 0.6)])
def test_counters_do_not_depend_on_the_path(n_cmax, boxes, spread):
    import paper_2511_21264_amd as mp
    ctx = mp.Context(0)
    sc = W.make_scene(5, n_box=boxes, n_cmax=n_cmax)
    scene, ext = mp.Scene(ctx, sc), mp.Scene(ctx, dict(sc, ext=1))
    K, H = 70, 5
    sig, nom = np.full(14, 0.3, np.float32), np.zeros((H, 14), np.float32)
    for i, x in enumerate(W.random_states(sc, 4, seed=2, spread=spread).astype(np.float32)):
        x[42:45] = [0.0, 0.0, sc["ball_r"] - 0.001 * (i % 2 == 0)]
        st = {}
        for m, s in (("wave", ext), ("split", ext), ("wave", scene), ("split", scene)):
            r = mp.mppi_plan(ctx, s, x, nom, K, H, 0.1, sig, np.zeros((H, 14), np.float32), np.zeros(K, np.float32),
                             M=1, seed=3, mapping=m)
            st[m, s is ext] = [r[k] for k in ("contacts", "np_tests", "box_tests", "overflow")]
        assert st["wave", True][1] > 0
        assert all(v == st["wave", True] for v in st.values()), st
    ctx.close()
