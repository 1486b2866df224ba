"""Rounds that score without the matrix-core filter (most residuals of sets of up
to 1,024 correspondences, or up to 32 candidates per query), which the library
picks by itself, against fixed launch shapes, which filter: the same bits in every
result.  Sizes lie on both sides of each line of the rule; batches mix sets on both
sides of it."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu

KEYS = ("candidates", "residuals", "inlier_residuals", "best_count", "best_msac", "best_h", "best_j", "final_cost")


def _same(a, b):
    assert list(a[0]) == list(b[0])
    for (Ra, ta), (Rb, tb) in zip(a[1], b[1]):
        np.testing.assert_array_equal(Ra, Rb)
        np.testing.assert_array_equal(ta, tb)
    for x, y in zip(a[2], b[2]):
        for k in KEYS:
            assert x[k] == y[k], k


@pytest.mark.parametrize("nq,sizes,samples", [
    (1, [512], 64), (1, [513], 64), (3, [1024], 25), (3, [1025], 25), (40, [2000], 24), (40, [2000], 25),
    (700, [512], 64), (700, [513], 256), (700, [1024], 64), (700, [1025], 64), (2100, [100], 16), (2100, [300], 200),
    (300, [100, 200, 5000], 64), (300, [900, 700, 1500], 128), (300, [400, 600, 3000], 30), (300, [3, 2, 5], 40)])
def test_batches(nq, sizes, samples):
    import paper_2601_04185_amd as pk
    base = [synth.make_query(820 + i, n, 0.4, 1.0, weights="conf") for i, n in enumerate(sizes)]
    ds = [pk.to_device(q) for q in base]
    k = len(base)
    prms = [pk.make_params(threshold_px=4.0, fixed_samples=samples, batch=samples, lo_top_k=2, query_id=i)
            for i in range(nq)]
    out = []
    for ct in (0, 64):
        ctx = pk.Context(0)
        ctx.set_score_tuning(ct, 0)
        out.append(pk.imloc_lo_ransac_pnp_batch(ctx, [ds[i % k] for i in range(nq)],
                                                [base[i % k].K for i in range(nq)], prms))
    _same(*out)


@pytest.mark.parametrize("n,count", [(512, 20000), (513, 9000), (1024, 3000), (1025, 3000), (5000, 32), (5000, 33),
                                     (300000, 31), (300000, 33)])
def test_given_poses(n, count):
    import torch
    import paper_2601_04185_amd as pk
    q = synth.make_query(830, n, 0.5, 1.0, weights="conf")
    d = pk.to_device(q)
    rng = np.random.default_rng(n)
    P = np.empty((count, 12))
    for i in range(count):
        P[i, :9] = (q.R if i % 2 else synth.random_rotation(rng)).ravel()
        P[i, 9:] = q.t + rng.normal(size=3) * (1e-3 if i % 2 else 2.0)
    P = torch.tensor(P, device="cuda")
    ref = None
    for ct in (64, 0, 128):
        ctx = pk.Context(0)
        ctx.set_score_tuning(ct, 0)
        cur = [x.cpu().numpy() for x in pk.imloc_score(ctx, d, q.K, P, 4.0, 0)]
        ref = ref or cur
        np.testing.assert_array_equal(cur[0], ref[0])
        np.testing.assert_array_equal(cur[1].view(np.int64), ref[1].view(np.int64))
    assert ref[0].max() > 0.4 * n
