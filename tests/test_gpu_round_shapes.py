"""The scoring launch shape that a round picks by itself (tile of 32 to 256
candidates, 512 to 2,048 correspondences per item) against fixed ones: per-
candidate sums are integers over fixed 512-wide blocks (Sec. 3.3 scoring), so
every result is the same bit for bit.  Sizes lie on both sides of each change of
the rule at 256 compute units, items counted at one candidate per sample."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,samples", [(3, 1), (600, 64), (6144, 1024), (6145, 1024), (16384, 1024), (16385, 1024),
                                       (40960, 1024), (38912, 1024), (98304, 1024), (96256, 1024), (2000, 4096)])
@pytest.mark.parametrize("weights", [False, True])
def test_round_shape_changes_nothing(n, samples, weights):
    import torch
    import paper_2601_04185_amd as pk
    q = synth.make_query(31, n, 0.4, 1.0)
    d = pk.to_device(q)
    d["w"] = torch.rand(n, generator=torch.Generator().manual_seed(n)).cuda() if weights else None
    prm = pk.make_params(threshold_px=4.0, fixed_samples=samples, batch=samples, lo_top_k=4)
    got = []
    for ct, pts in ((0, 2048), (0, 512), (32, 2048), (128, 2048)):
        ctx = pk.Context(0)
        ctx.set_score_tuning(ct, 0)
        ctx.set_score_points(pts)
        assert ctx.score_tuning() == (ct, 0) and ctx.score_points() == pts
        got.append(pk.imloc_lo_ransac_pnp(ctx, d, q.K, prm))
        assert ctx.score_points() == pts
    for rc, R, t, st in got[1:]:
        assert rc == got[0][0]
        np.testing.assert_array_equal(R, got[0][1])
        np.testing.assert_array_equal(t, got[0][2])
        for k in ("candidates", "residuals", "inlier_residuals", "best_count", "best_msac", "best_h", "best_j"):
            assert st[k] == got[0][3][k], k
