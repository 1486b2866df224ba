"""Batches of more queries than one look of a Gauss-Newton workgroup holds: it
finds its query by 256 first tickets a step, one step up to 256 queries, two up
to 65,536.  A query's result is that of the query alone, bit for bit; teams of one
and of several workgroups alternate, so that the tickets are not the queries'
numbers."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq", [2, 255, 256, 257, 511, 513, 4099, 65535])
def test_each_query_as_alone(nq):
    import paper_2601_04185_amd as pk
    ctx = pk.Context(0)
    base = [synth.make_query(600 + i, 2100 if i % 3 == 1 and nq < 10000 else 60 + i, 0.5, 1.0) for i in range(7)]
    ds = [pk.to_device(q) for q in base]
    prms = [pk.make_params(threshold_px=4.0, fixed_samples=16, batch=16, lo_top_k=1 + i % 2, query_id=i % 97)
            for i in range(nq)]
    many = pk.imloc_lo_ransac_pnp_batch(ctx, [ds[i % 7] for i in range(nq)], [base[i % 7].K for i in range(nq)], prms)
    alone = pk.Context(0)
    look = {0, 1, nq // 2, nq - 2, nq - 1} | set(range(0, nq, max(1, nq // 12))) | {255, 256, 257, 512, 65280}
    for i in sorted(i for i in look if i < nq):
        rc, R, t, st = pk.imloc_lo_ransac_pnp(alone, ds[i % 7], base[i % 7].K, prms[i])
        assert rc == many[0][i], i
        np.testing.assert_array_equal(R, many[1][i][0], err_msg=str(i))
        np.testing.assert_array_equal(t, many[1][i][1], err_msg=str(i))
        for k in ("best_h", "best_j", "best_msac", "final_cost", "full_count", "lo_runs"):
            assert st[k] == many[2][i][k], (i, k)
