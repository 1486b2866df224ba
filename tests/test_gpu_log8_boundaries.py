"""The log-depth encoder where its float32 level cannot decide: depths on both
sides of every rounding boundary, from neighbouring floats out to where the
float32 level takes over, against the oracle's float64 encoder (bit-exact).
Lengths around a workgroup's 4,096 entries, at an aligned and an unaligned
address."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("n", [1, 7, 4095, 4096, 4097, 8195, 254 * 121])
def test_encode_at_every_boundary(orc, n, shift):
    import torch
    import paper_2601_04185_amd as pk
    b = 0.25 * 512.0 ** ((np.arange(1, 255) - 0.5) / 254.0)  # between codes c and c + 1
    at = b.astype(np.float32).view(np.int32)
    near = np.arange(-20, 21)                                # floats around the boundary,
    far = np.round(1.35 ** np.arange(8, 48)).astype(np.int64)  # then out to half a level
    off = np.concatenate([near, far, -far])
    assert len(off) == 121
    d = (at[None, :] + off[:, None]).astype(np.int32).view(np.float32).reshape(-1)[:n]
    buf = torch.from_numpy(np.concatenate([np.full(shift, 1.0, np.float32), d])).cuda()
    got = pk.imloc_depth_encode_log8(pk.Context(0), buf[shift:]).cpu().numpy()
    np.testing.assert_array_equal(got, orc.log8_encode(d))
