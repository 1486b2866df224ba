"""Depth by triangulation at the sizes where its launches change shape, against
the float64 oracle, with the bar of test_gpu_triangulate.py: view counts around
the groups of hypotheses (5), of loads (16), the workgroups' LDS limit (14, 15
and 28, 29 views) and the members a lane keeps (multiples of 4); angular
thresholds below and beyond the angle where the refinement leaves its series
for atan2 (5.7 degrees); a view that is the mapping view itself, whose rays
tell nothing."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth
from test_gpu_triangulate import _check, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("angle", [2.0, 9.0, 25.0])
@pytest.mark.parametrize("V,H,W", [(4, 16, 16), (5, 17, 31), (6, 15, 17), (14, 16, 17), (15, 9, 29), (28, 8, 16),
                                   (29, 7, 19)])
def test_parity_at_launch_edges(orc, V, H, W, angle):
    import paper_2601_04185_amd as pk
    w = synth.dense_match_scene(n_views=V, width=W, height=H, correct_frac=0.8, noise_px=0.3, seed=60 + V, f=0.8 * 96)
    w.Ts[V // 2] = w.T0
    w.Ks[V // 2] = w.K0
    j, i = np.meshgrid(np.arange(W) + 0.5, np.arange(H) + 0.5)
    w.mu[V // 2], w.mv[V // 2] = j, i
    g = _run(pk, pk.Context(0), w, angle_deg=angle)
    r = orc.triangulate(w.K0, w.T0, w.Ks, w.Ts, w.mu, w.mv, w.conf, angle_deg=angle)
    _check(g, r, max_flagged=0.05, min_inliers=3)
