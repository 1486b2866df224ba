"""Lifting in one launch at the sizes where its tiles (1,024 matches) and its
window of earlier tiles (256) end, against the oracle: the same matches kept in
the same order (bit-exact source indices), world points within one float32 ulp
of the oracle's float64.  Forms: waiting for the counts of the tiles before;
counting them alone (zero polls, set from the host); with a host staging buffer
that has no room for the zeroed counts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _inputs(n, codes, rng):
    nv, H, W = 3, 37, 53
    f = lambda lo, hi, k: rng.uniform(lo, hi, k).astype(np.float32)
    depth = f(0.5, 30.0, (nv, H, W))
    if codes:
        depth = rng.integers(1, 256, (nv, H, W)).astype(np.uint8)
    depth[rng.random(depth.shape) < 0.02] = 0
    m = dict(q_u=f(0, 640, n), q_v=f(0, 480, n), db_u=f(-1, W + 1, n), db_v=f(-1, H + 1, n), conf=f(0, 1, n),
             view=rng.integers(-1, nv + 1, n).astype(np.int32))
    if n > 3000:  # whole tiles that keep nothing, and whole tiles that keep what they can
        m["conf"][1024:2048] = 0.0
        m["conf"][2048:3072] = 1.0
    cams = np.tile(np.array((500.0, 510.0, 26.0, 18.0)), (nv, 1))
    q = np.linalg.qr(rng.normal(size=(nv, 3, 3)))[0]
    poses = np.concatenate([q.reshape(nv, 9), rng.normal(size=(nv, 3))], 1)
    return m, depth, cams, poses


@pytest.mark.parametrize("codes,subpixel", [(False, True), (True, True), (True, False)])
@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 2049, 5000, 256 * 1024 + 1, 258 * 1024])
def test_lift_tiles(orc, n, codes, subpixel):
    import torch
    import paper_2601_04185_amd as pk
    m, depth, cams, poses = _inputs(n, codes, np.random.default_rng(n + 3 * codes + subpixel))
    dm = {k: torch.from_numpy(v).cuda() for k, v in m.items()}
    ref = orc.lift(m, depth, cams, poses, subpixel=subpixel)
    for form in ("wait", "alone", "small_staging"):
        ctx = pk.Context(0)
        if form == "alone":
            ctx.check(pk.lib().gn_set_team_polls(ctx.h, 0))
        if form == "small_staging":
            ctx.check(pk.lib().imloc_set_staging(ctx.h, 16 * 8 * len(cams) + 512))
        for cap in (None, max(1, len(ref["src"]) - 7)):
            g = pk.imloc_lift(ctx, dm, torch.from_numpy(depth).cuda(), cams, poses, subpixel=subpixel, capacity=cap)
            k = len(ref["src"]) if cap is None else min(cap, len(ref["src"]))
            assert g["n"] == len(ref["src"]) and g["src"].numel() == k, form
            np.testing.assert_array_equal(g["src"].cpu().numpy(), ref["src"][:k], err_msg=form)
            for c in ("u", "v", "w"):
                np.testing.assert_array_equal(g[c].cpu().numpy(), ref[c][:k].astype(np.float32))
            for c in ("X", "Y", "Z"):
                b = ref[c][:k]
                tol = 1.01 * np.spacing(np.abs(b).astype(np.float32)).astype(np.float64) + 1e-12
                assert np.all(np.abs(g[c].cpu().numpy().astype(np.float64) - b) <= tol), form
