"""Matches given as strided views: the binding's contiguous copies stay alive while
the workspace is allocated, which would otherwise take their memory."""
import numpy as np
import pytest

from paper_2601_04185_amd import synth

pytestmark = pytest.mark.gpu


def test_strided_matches():
    import torch
    import paper_2601_04185_amd as pk
    w = synth.dense_match_scene(n_views=6, width=96, height=80)
    m = [torch.as_tensor(np.asarray(a, np.float32), device="cuda") for a in (w.mu, w.mv, w.conf)]
    want = pk.imloc_triangulate_depth(pk.Context(0), w.K0, w.T0, w.Ks, w.Ts, *m, want_codes=True)
    strided = [a.permute(1, 2, 0).contiguous().permute(2, 0, 1) for a in m]
    assert not strided[0].is_contiguous()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    for _ in range(3):  # a new context has no workspace yet
        got = pk.imloc_triangulate_depth(pk.Context(0), w.K0, w.T0, w.Ks, w.Ts, *strided, want_codes=True)
        for k in ("depth", "inliers", "codes"):
            assert torch.equal(got[k], want[k]), k
