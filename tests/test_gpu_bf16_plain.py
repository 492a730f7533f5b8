"""polydl_conv2d_fwd_bf16 blocks input and filter in one launch where it can: same bits as the blocked entry
points, whatever the sizes of the two tensors against each other."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [
    synth.ConvShape("tiny_image_big_filter", 1, 20, 4, 4, 300, 3, 3, 1, 1),       # filter slices behind one image
    synth.ConvShape("one_unit", 2, 3, 8, 8, 1, 1, 1, 1, 0),                        # one filter unit
    synth.ConvShape("ragged_channels", 3, 37, 8, 6, 65, 1, 1, 1, 0),
    synth.ConvShape("two_pixel_blocks", 2, 64, 24, 24, 33, 5, 5, 1, 2),            # 576 pixels: two blocks of 512
    synth.ConvShape("narrow", 2, 16, 7, 5, 24, 3, 3, 1, 1),                        # H*W no multiple of 8: two launches
], ids=lambda s: s.name)
def test_plain_equals_blocked(s):
    import torch
    import paper_2006_02230_amd as P
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x, w, b = synth.conv_inputs(s, seed=9, dist="normal", bias=True)
    x = torch.from_numpy(x).cuda().to(torch.bfloat16)
    w = torch.from_numpy(w).cuda().to(torch.bfloat16)
    b = torch.from_numpy(b).cuda()
    got = P.conv2d_fwd_bf16(x, w, b, stride=s.stride, pad=s.pad, act="relu")
    want = P.conv2d_fwd_bf16_blocked(P.nchw_to_nchwc_bf16(x, 8), P.kcrs_to_kcrsck_bf16(w, 8, 1), s.C, b, stride=s.stride, pad=s.pad,
                                     act="relu")
    assert np.array_equal(got.cpu().numpy(), want.cpu().numpy())
