"""A query's candidates are shared out alike over the tiles of its scoring (not
full tiles and a rest).  Scores are sums of integers per candidate, so the
results are those of other tiles bit for bit; the numbers of candidates lie
around one, two and three tiles of 32, 128 and 256, float64 items share the cut."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu

COUNTS = [1, 31, 32, 33, 64, 65, 97, 127, 128, 129, 161, 255, 256, 257, 289, 350, 511, 512, 513, 700, 769, 1025]


@pytest.mark.parametrize("precision", [0, 1])
def test_numbers_of_candidates(precision):
    import torch
    import paper_2601_04185_amd as pk
    q = synth.make_query(991, 3000, 0.6, 1.0, weights="conf")
    d = pk.to_device(q)
    rng = np.random.default_rng(3)
    P = np.empty((max(COUNTS), 12))
    for i in range(len(P)):
        P[i, :9] = (q.R if i % 3 == 0 else synth.random_rotation(rng)).ravel()
        P[i, 9:] = q.t + rng.normal(size=3) * (1e-3 if i % 3 == 0 else 2.0)
    P = torch.tensor(P, device="cuda")
    ref = [x.cpu().numpy() for x in pk.imloc_score(pk.Context(0), d, q.K, P, 4.0, precision)]
    assert ref[0].max() > 1000
    for ct in (0, 32, 64, 128):
        ctx = pk.Context(0)
        ctx.set_score_tuning(ct, 0)
        for n in COUNTS:
            cnt, ms = (x.cpu().numpy() for x in pk.imloc_score(ctx, d, q.K, P[:n].contiguous(), 4.0, precision))
            np.testing.assert_array_equal(cnt, ref[0][:n], err_msg=str((ct, n)))
            np.testing.assert_array_equal(ms.view(np.int64), ref[1][:n].view(np.int64), err_msg=str((ct, n)))


def test_batch_of_two_tiles():
    """2,100 queries of about 350 candidates (two tiles of up to 256) each as alone."""
    import paper_2601_04185_amd as pk
    ctx, alone = pk.Context(0), pk.Context(0)
    alone.set_score_tuning(32, 0)
    qs = [synth.make_query(700 + i, 2000, 0.3, 1.0) for i in range(5)]
    ds = [pk.to_device(q) for q in qs]
    nq = 2100
    prms = [pk.make_params(threshold_px=4.0, fixed_samples=256, batch=256, lo_top_k=2, query_id=i) for i in range(nq)]
    many = pk.imloc_lo_ransac_pnp_batch(ctx, [ds[i % 5] for i in range(nq)], [qs[i % 5].K for i in range(nq)], prms)
    for i in range(0, nq, 150):
        rc, R, t, st = pk.imloc_lo_ransac_pnp(alone, ds[i % 5], qs[i % 5].K, prms[i])
        assert rc == many[0][i] and st["candidates"] > 256
        np.testing.assert_array_equal(R, many[1][i][0])
        np.testing.assert_array_equal(t, many[1][i][1])
        for k in ("best_h", "best_j", "best_msac", "inlier_residuals", "candidates"):
            assert st[k] == many[2][i][k], (i, k)
