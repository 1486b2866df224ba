"""Rig queries whose cameras' points begin inside the groups that the Gauss-Newton
runs cut a problem into: groups of one, two and many cameras, cameras without a
point or with one.  A group whose points are read from memory (one workgroup per
problem) takes each point's camera from the starts of the group's first two; one
kept in LDS (the widest team) looked it up once; both must give the same bits."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


def _uneven(sizes, seed):
    """A rig query with the given number of points per camera."""
    q = synth.make_rig_query(seed, len(sizes) * max(sizes), 0.6, 1.0, n_cams=len(sizes))
    start = q.cam_start()
    keep = np.concatenate([np.arange(start[c], start[c] + s) for c, s in enumerate(sizes)]).astype(np.int64)
    a = [np.ascontiguousarray(x[keep]) for x in (q.u, q.v, q.X, q.Y, q.Z)]
    return synth.RigQuery(*a, None, q.cam[keep], q.rig, q.R, q.t, q.is_inlier[keep])


@pytest.mark.parametrize("sizes", [(2500, 2500), (1, 3000), (3000, 1), (2048, 1024, 1025), (5, 1000, 3, 2000, 7, 1, 4000, 900),
                                   (0, 1500, 0, 0, 1500, 2), (30000, 40, 30000, 200, 9000, 1, 0, 2000)])
def test_cameras_inside_groups(sizes):
    import torch
    import paper_2601_04185_amd as pk
    q = _uneven(sizes, 870 + len(sizes))
    d = pk.to_device(q)
    prm = pk.make_params(threshold_px=4.0, fixed_samples=300, batch=300, lo_top_k=3)
    out = []
    for mode in (1, 2):
        ctx = pk.Context(0)
        ctx.set_gn_mode(mode)
        mask = torch.full((q.n,), 7, dtype=torch.uint8, device="cuda")
        rc, R, t, st = pk.imloc_rig_lo_ransac_pnp(ctx, d, q.rig, q.cam_start(), prm, mask)
        out.append([rc, R, t, st["best_msac"], st["final_cost"], st["full_count"], mask.cpu().numpy()])
    assert out[0][0] == 0 and out[0][5] > 0.4 * q.n
    for a, b in zip(*out):
        np.testing.assert_array_equal(a, b)
