"""The top-k choice among generalised P3P candidates (Sec. 3.3 "Pose
Estimation"): a sample has up to eight solutions, and without a good pose most
candidates see their own three points alone, so that their costs tie and the
sample and the solution decide.  The chosen ones are those of a sort on the host
of the scores that the scoring stage gives for the sampling stage's candidates.
Without Gauss-Newton iterations a run returns one of the chosen poses as it was
(exact match): the first for k = 1, any of the first k otherwise, and k runs are
counted."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


def _three_cameras(seed, spread):
    """A point in each of three cameras `spread` metres apart: every sample is
    the same triple, and wide rigs have triples with five and six solutions
    (one of the seeds' rigs in a thousand)."""
    rng = np.random.default_rng(seed)
    K = (380.0, 380.0, 320.0, 240.0)
    rig, px, X = [], [], []
    for _ in range(3):
        Rc, c = synth.random_rotation(rng), rng.normal(size=3) * spread
        rig.append((K, np.concatenate([Rc.reshape(9), -Rc @ c])))
        p, z = rng.random(2) * np.array([640, 480]), rng.uniform(2, 20)
        px.append(p)
        X.append(Rc.T @ np.array([(p[0] - K[2]) / K[0] * z, (p[1] - K[3]) / K[1] * z, z]) + c)
    px, X = np.array(px, np.float32), np.array(X, np.float32)
    a = [np.ascontiguousarray(v) for v in (px[:, 0], px[:, 1], X[:, 0], X[:, 1], X[:, 2])]
    return synth.RigQuery(*a, None, np.arange(3, dtype=np.int32), rig, np.eye(3), np.zeros(3), np.zeros(3, bool))


def _check(q, samples, precision, ks):
    import paper_2601_04185_amd as pk
    ctx = pk.Context(0)
    d = pk.to_device(q)
    g = pk.imloc_rig_sample_gp3p(ctx, d, q.rig, q.cam_start(), seed=0, query_id=0, h0=0, count=samples)
    h, j, poses = (g[k].cpu().numpy() for k in ("h", "j", "poses"))
    cnt, ms = (x.cpu().numpy() for x in pk.imloc_rig_score(ctx, d, q.rig, q.cam_start(), g["poses"], 4.0, precision))
    order = np.lexsort((j, h, -cnt.astype(np.int64), ms))
    for k in ks:
        prm = pk.make_params(threshold_px=4.0, fixed_samples=samples, batch=samples, lo_top_k=k, lo_iters=0,
                             final_iters=0, precision=precision)
        rc, R, t, st = pk.imloc_rig_lo_ransac_pnp(ctx, d, q.rig, q.cam_start(), prm)
        assert rc == 0 and st["candidates"] == len(h) and st["lo_runs"] == min(k, len(h))
        hit = [i for i in order[:k] if (h[i], j[i]) == (st["best_h"], st["best_j"])]
        assert len(hit) == 1, (k, st["best_h"], st["best_j"])
        np.testing.assert_array_equal(np.concatenate([R.reshape(9), t]), poses[hit[0]])
    return h[order], j[order], cnt[order], ms[order]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("seed,spread,solutions", [(1443, 10, 5), (4633, 10, 5), (4362, 10, 6), (5244, 10, 6),
                                                   (1156, 20, 6)])
def test_more_than_four_solutions(seed, spread, solutions, precision):
    q = _three_cameras(seed, spread)
    h, j, cnt, ms = _check(q, 16, precision, range(1, 9))
    # (sample 0 draws no three different points)
    assert j.max() == solutions - 1 and len(h) == 15 * solutions
    if precision == 1:  # the fifth solution of one sample and the first of the next cost the same
        assert len(set(zip(h[:8] * 4 + j[:8], cnt[:8], ms[:8]))) < 8


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("samples", [64, 4096])
def test_no_good_pose(samples, precision):
    """Outliers alone, in one workgroup and in several."""
    _check(synth.make_rig_query(57, 60, 0.0, 1.0), samples, precision, (1, 7, 8, 9))
