"""Float32 scoring with the matrix-core filter against scoring without it.

Work items of 32 candidates x 512 correspondences give each wave 8 candidates,
too few for the filter, so they evaluate every residual; every other shape
filters from 12 candidates on.  Counts and truncated costs must be the same
bits (no tolerance): the filter only leaves out what holds no inlier.  Sizes
are the edges of the 32-wide products, the 64-wide slots, the 512-wide blocks
and the 256-candidate tile; inputs hold what a float16 bound could get wrong:
no spread at all, spreads of very different size, far offsets, values out of
float32's or float16's range, infinities and NaN."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


def _poses_around(rng, q, count):
    import torch
    out = np.empty((count, 12))
    for i in range(count):
        R, t = (q.R, q.t) if i % 3 == 0 else (synth.random_rotation(rng), synth.random_translation(rng, 5.0))
        w = rng.normal(size=3) * 10.0 ** rng.uniform(-5, -1)
        dR = np.eye(3) + np.array([[0, -w[2], w[1]], [w[2], 0, -w[0]], [-w[1], w[0], 0]])
        u, _, vt = np.linalg.svd(dR @ R)
        out[i, :9] = (u @ vt).reshape(-1)
        out[i, 9:] = t + rng.normal(size=3) * 10.0 ** rng.uniform(-4, 0)
    return torch.tensor(out, device="cuda")


def _change(form, c, rng, K):
    X = np.stack([c["X"], c["Y"], c["Z"]], 1).astype(np.float64)
    n = len(X)
    if form == "one_point":
        for k in ("u", "v", "X", "Y", "Z"):
            c[k][:] = c[k][0]
    elif form == "flat":
        c["Z"][:] = c["Z"][0]
    elif form == "far":
        for k in ("X", "Y", "Z"):
            c[k] += np.float32(3e4)
    elif form == "uneven":
        c["X"][rng.integers(n, size=max(1, n // 50))] = 1e6
        c["u"][rng.integers(n, size=max(1, n // 50))] = -1e5
    elif form == "huge":
        c["Y"][rng.integers(n, size=max(1, n // 300))] = 3e38
        c["v"][rng.integers(n, size=max(1, n // 300))] = -3e38
    elif form == "odd":
        for k, x in (("X", np.nan), ("Z", np.inf), ("u", -np.inf), ("v", np.nan)):
            c[k][rng.integers(n, size=max(1, n // 200))] = x
    elif form == "tiny":
        for k in ("X", "Y", "Z"):
            c[k] *= np.float32(1e-30)


@pytest.mark.parametrize("form", ["plain", "one_point", "flat", "far", "uneven", "huge", "odd", "tiny"])
@pytest.mark.parametrize("n,count", [(1, 12), (63, 31), (64, 32), (511, 33), (513, 11), (2049, 65), (2560, 257),
                                     (6000, 300), (140000, 7700)])
def test_filter_changes_no_bit(form, n, count):
    import torch
    import paper_2601_04185_amd as pk
    if n > 10000 and form not in ("plain", "odd"):
        pytest.skip("large sizes: two forms")
    rng = np.random.default_rng(31 * n + len(form))
    q = synth.make_query(900 + n, n, 0.3, 1.0, weights="conf")
    c = {k: (None if v is None else np.array(v, np.float32)) for k, v in q.corr().items()}
    _change(form, c, rng, q.K)
    dev = {k: torch.tensor(v, device="cuda") for k, v in c.items()}
    poses = _poses_around(rng, q, count)
    if form == "far":  # keeps a third of the candidates on their inliers
        R = poses[:, :9].reshape(-1, 3, 3)
        poses[:, 9:] -= R @ torch.full((3,), 3e4, device="cuda", dtype=torch.float64)
    poses = poses.contiguous()
    ref = None
    for ct, pts in [(32, 512), (0, 2048), (32, 2048), (64, 1024), (64, 4096), (128, 512), (128, 2048)]:
        ctx = pk.Context(0)
        ctx.set_score_tuning(ct, 0)
        ctx.set_score_points(pts)
        cur = [x.cpu().numpy() for x in pk.imloc_score(ctx, dev, q.K, poses, 4.0, 0)]
        if ref is None:
            ref = cur
            if form == "plain" and n > 60:
                assert ref[0].max() > 0.1 * n  # (there is something to find)
        np.testing.assert_array_equal(cur[0], ref[0], err_msg=str((ct, pts)))
        np.testing.assert_array_equal(cur[1].view(np.int64), ref[1].view(np.int64), err_msg=str((ct, pts)))
