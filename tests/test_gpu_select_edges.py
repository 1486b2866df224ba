"""The top-k choice at the edges of its work split (Sec. 3.3 "Pose Estimation"):
1,024 candidates per workgroup, at most 8 workgroups per query, fewer per
query the more queries a launch has.  Most poses see no inlier at all, so
their costs tie and the index decides (a strict total order: exact match)."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 7, 64, 1023, 1024, 1025, 2049, 8192, 8193, 17000])
def test_select_edges(count):
    import torch
    import paper_2601_04185_amd as pk
    ctx = pk.Context(0)
    q = synth.make_query(4243, 600, 0.3, 1.0)
    d = pk.to_device(q)
    rng = np.random.default_rng(count)
    poses = np.zeros((count, 12))
    for i in range(count):
        near = i % 97 == 3
        R = q.R if near else synth.random_rotation(rng)
        poses[i, :9] = R.ravel()
        poses[i, 9:] = q.t + rng.normal(size=3) * (0.02 if near else 50.0)
    P = torch.tensor(poses, dtype=torch.float64, device="cuda")
    cnt, ms = (x.cpu().numpy() for x in pk.imloc_score(ctx, d, q.K, P, 4.0))
    order = np.lexsort((np.arange(count), -cnt.astype(np.int64), ms))
    for k in (1, 5, 8):
        for gate in (float("inf"), float(np.nextafter(ms[order[min(count, 4) - 1]], np.inf)), float(ms.max())):
            want = [i for i in order if ms[i] < gate][:k]
            got = pk.imloc_select_top_k(ctx, d, q.K, P, 4.0, k, gate).cpu().numpy()
            assert list(got) == want, (count, k, gate)


@pytest.mark.parametrize("nq", [33, 256])
def test_select_many_queries_equals_alone(nq):
    """A query's candidates in one workgroup (256 queries), in up to 7 (33) and in up to 8 (alone)."""
    import paper_2601_04185_amd as pk
    ctx = pk.Context(0)
    qs = [synth.make_query(900 + i, 40 + i, 0.3, 1.0) for i in range(nq)]
    ds = [pk.to_device(q) for q in qs]
    prms = [pk.make_params(threshold_px=4.0, fixed_samples=5000, batch=5000, lo_top_k=8, query_id=i)
            for i in range(nq)]
    many = pk.imloc_lo_ransac_pnp_batch(ctx, pk.BatchQueries(ds, [q.K for q in qs], prms))
    for i in range(0, nq, 16):
        rc, R, t, st = pk.imloc_lo_ransac_pnp(ctx, ds[i], qs[i].K, prms[i])
        assert st["candidates"] > 2048 and rc == many[0][i]
        np.testing.assert_array_equal(R, many[1][i][0])
        np.testing.assert_array_equal(t, many[1][i][1])
        assert (st["best_h"], st["best_j"]) == (many[2][i]["best_h"], many[2][i]["best_j"])
