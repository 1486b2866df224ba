"""The weight sum of a small scoring set after that of a large one in the same
workspace: the parts past its end are zero, not what the large set left there.
A pose with every point behind the camera costs tau^2 times the sum (float64, at
most 64 additions per thread and 30 more: 1e-13 relative)."""
import math

import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


def test_sizes_in_one_workspace():
    import torch
    import paper_2601_04185_amd as pk
    ctx = pk.Context(0)
    for n in (40000, 1, 1024, 20000, 1025, 2048, 2049, 15361, 5, 16384, 300):
        q = synth.make_query(72, n, 0.4, 1.0)
        w = np.random.default_rng(n).uniform(0.05, 1.0, n).astype(np.float32)
        d = dict(pk.to_device(q), w=torch.from_numpy(w).cuda())
        pose = torch.tensor(np.concatenate([q.R.ravel(), [0.0, 0.0, -1e4]])[None], device="cuda")
        cnt, ms = pk.imloc_score(ctx, d, q.K, pose, 3.0)
        want = 9.0 * math.fsum(w.astype(np.float64))
        assert int(cnt[0]) == 0 and abs(float(ms[0]) - want) <= 1e-13 * want, n
