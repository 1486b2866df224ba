"""Teams of the Gauss-Newton runs: a problem's groups of points are shared by
workgroups that exchange their sums inside one launch.  The sums and their
order depend on the problem alone, so a result must be bitwise the same for one
workgroup per problem, for the widest team, and for members that do not wait
for the others at all but evaluate every group themselves (the bounded wait of
a member set to zero polls from the host), at the sizes where the cut into
groups changes: one group, two, one point in the last one, 32 groups, groups of
2,048 and of 4,096 points."""
import ctypes as C

import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu

FORMS = ((2, None), (1, None), (1, 0), (0, 0))  # team mode, polls of a wait


@pytest.fixture(scope="module")
def pk():
    import torch
    import paper_2601_04185_amd as pk
    assert torch.cuda.is_available()
    f = pk.lib().gn_set_team_polls
    f.argtypes, f.restype = [C.c_void_p, C.c_int32], C.c_int
    return pk


def _ctx(pk, mode, polls):
    ctx = pk.Context(0)
    ctx.set_gn_mode(mode)
    if polls is not None:
        ctx.check(pk.lib().gn_set_team_polls(ctx.h, polls))
    return ctx


def _starts(q, k, seed):
    rng = np.random.default_rng(seed)
    P = np.tile(np.concatenate([q.R.reshape(9), q.t]), (k, 1))
    P[:, 9:] += rng.normal(0, 0.03, (k, 3))
    return P


@pytest.mark.parametrize("n", [3, 255, 2048, 2049, 3073, 32768, 32769, 65537, 131073, 262145])
def test_stages_do_not_depend_on_the_team(pk, n):
    import torch
    q = synth.make_query(940 + n % 89, n, 0.5, 1.0, weights="conf")
    d = pk.to_device(q)
    start = torch.from_numpy(_starts(q, 3, n)).cuda()
    out = []
    for mode, polls in FORMS:
        ctx = _ctx(pk, mode, polls)
        mask = torch.full((n,), 7, dtype=torch.uint8, device="cuda")
        got = list(pk.imloc_local_optimize(ctx, d, q.K, start, 4.0, iters=10))
        got += list(pk.imloc_refine(ctx, d, q.K, start[0].contiguous(), 4.0, 2.0, iters=10, mask=mask)) + [mask]
        out.append([t.cpu().numpy() for t in got])
    for form, other in zip(FORMS[1:], out[1:]):
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b, equal_nan=a.dtype.kind == "f"), form


def test_queries_do_not_depend_on_the_team(pk):
    """Two rounds of two queries and a rig query (mailboxes are used again in
    the second round), with the mask of the final pose."""
    import torch
    qs = [synth.make_query(960 + i, n, 0.3, 1.0) for i, n in enumerate([5000, 40000])]
    P = [pk.make_params(threshold_px=4.0, fixed_samples=1024, batch=512, lo_top_k=4, query_id=i) for i in range(2)]
    rig = synth.make_rig_query(965, 6000, 0.4, 1.0)
    out = []
    for mode, polls in FORMS:
        ctx = _ctx(pk, mode, polls)
        masks = [torch.full((q.n,), 7, dtype=torch.uint8, device="cuda") for q in qs + [rig]]
        st, poses, stats = pk.imloc_lo_ransac_pnp_batch(ctx, [pk.to_device(q) for q in qs], [q.K for q in qs], P,
                                                        masks=masks[:2], arrays=True)
        r = pk.imloc_rig_lo_ransac_pnp(ctx, pk.to_device(rig), rig.rig, rig.cam_start(), P[0], masks[2])
        assert list(st) == [0, 0] and r[0] == 0
        out.append([poses, stats["best_msac"], stats["final_cost"], stats["full_count"], r[1], r[2],
                    np.float64(r[3]["final_cost"])] + [m.cpu().numpy() for m in masks])
    for form, other in zip(FORMS[1:], out[1:]):
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b), form
