"""Short reductions into at most 64 output channels (first layers), with enough pixels for the kernel that keeps the whole
split filter in LDS: edges of its units, steps and tap masks against the oracle."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import FP32_TOL, dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_02230_amd as p
    p.set_tile_override(None)
    yield p


# 98304 pixels (1536 units of 64) and more take the kernel on a card of 256 compute units
SHAPES = [synth.ConvShape("first_layer", 2, 3, 450, 451, 64, 7, 7, 2, 3),        # odd rows, a last unit of 4 pixels
          synth.ConvShape("two_steps", 1, 3, 320, 321, 50, 3, 3, 1, 1),          # 27 rows
          synth.ConvShape("63_taps", 1, 6, 318, 331, 33, 7, 9, 1, 4),            # every mask bit; 378 rows, the longest
          synth.ConvShape("strided_45_taps", 3, 4, 560, 549, 64, 5, 9, 3, 3),
          synth.ConvShape("no_padding", 4, 8, 161, 163, 64, 3, 3, 1, 0),
          synth.ConvShape("small_images", 2100, 5, 7, 7, 17, 3, 3, 1, 1),        # a unit touches three images
          synth.ConvShape("1x1", 40, 131, 50, 50, 64, 1, 1, 1, 0),
          synth.ConvShape("1x1_strided_padded", 11, 130, 190, 191, 20, 1, 1, 2, 1),
          synth.ConvShape("one_unit_less", 24, 16, 64, 64, 64, 3, 3, 1, 1),      # 1536 units; 23 images: the picked tile
          synth.ConvShape("below", 23, 16, 64, 64, 64, 3, 3, 1, 1)]


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: s.name)
def test_against_the_oracle(P, s):
    x, w, b = synth.conv_inputs(s, seed=3 + len(s.name), dist="normal", bias=True)
    dx, dw, db = dev(x), dev(w), dev(b)
    for act, bias, pre in (("relu6", True, None), ("none", False, "relu")):
        want, ab = oracle.conv2d_fwd(np.maximum(x, 0) if pre else x, w, bias=b if bias else None, stride=s.stride, pad=s.pad, act=act)
        got = host(P.conv2d_fwd(dx, dw, db if bias else None, stride=s.stride, pad=s.pad, act=act, pre_act=pre))
        assert oracle.scaled_error(got, want, ab) <= FP32_TOL, (act, pre)


@pytest.mark.parametrize("case", ["inf", "nan_filter", "lowest", "tiny", "tiny_filter"])
def test_values_the_split_cannot_hold(P, case):
    s = synth.ConvShape("v", 3, 3, 381, 379, 60, 5, 5, 2, 2)
    x, w, _ = synth.conv_inputs(s, seed=5, dist="normal")
    if case == "inf":
        x[1, 2, 0, 378] = np.inf
    elif case == "nan_filter":
        w[7, 1, 2, 0] = np.nan
    elif case == "lowest":
        x[0, 1, 3, 3] = np.finfo(np.float32).min
        w *= np.float32(1e-3)
    elif case == "tiny":
        x[2, :, 100:] *= np.float32(1e-37)
        w *= np.float32(1e20)
    elif case == "tiny_filter":
        w[40] *= np.float32(1e-37)
        x *= np.float32(1e20)
    # the padding is zeros that are multiplied like any other value
    want, ab = oracle.conv2d_fwd(np.pad(x, ((0, 0), (0, 0), (s.pad, s.pad), (s.pad, s.pad))), w, stride=s.stride, pad=0)
    got = host(P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad))
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[~fin], want[~fin].astype(np.float32), equal_nan=True)
    # 75 sequential roundings where a unit is recomputed with fp32 instructions, the last one of the store
    assert (np.abs(got[fin] - want[fin]) <= (75 + 2) * 2.0 ** -24 * ab[fin]).all()


def test_short_reduction_into_many_channels(P):
    # the fp32 gather kernel with its row table on a grid that fills the card: padding at every image border reads as zero
    s = synth.ConvShape("b", 64, 3, 28, 15, 512, 5, 5, 1, 2)
    x, w, b = synth.conv_inputs(s, seed=9, dist="normal", bias=True)
    want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad)
    dx, dw, db = dev(x), dev(w), dev(b)
    for _ in range(4):
        assert oracle.scaled_error(host(P.conv2d_fwd(dx, dw, db, stride=s.stride, pad=s.pad)), want, ab) <= FP32_TOL


THIN = dict(bm=64, bn=64, bk=0, wm=64, wn=64, split_k=1, layout=0, raster=0, algo=3, cb=0)


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: s.name)
def test_the_kernel_that_ran_is_reported(P, s):
    x, w, _ = synth.conv_inputs(s, seed=4, dist="normal")
    dx, dw = dev(x), dev(w)
    first = P.conv2d_fwd(dx, dw, stride=s.stride, pad=s.pad)
    ran = P.get_last_tile()
    if s.name == "below":
        assert ran.algo != 3
    else:
        assert ran.as_dict() == THIN
    # what is reported can be forced, modelled, and gives the same bits
    assert P.model_conv2d(tuple(s)[1:], ran).predicted_us > 0
    P.set_tile_override(ran)
    assert (P.conv2d_fwd(dx, dw, stride=s.stride, pad=s.pad) == first).all()
    assert P.get_last_tile().as_dict() == ran.as_dict()
    P.set_tile_override(None)


# reductions of up to 80 rows: where more than 45 % (up to 48 rows; else 55 %) of what the kernel multiplies is not the layer's, the
# picked tile is the faster one; (C, H, W, N, K, R, S, stride), with compute units' waves of 2048
@pytest.mark.parametrize("C,H,W,N,K,R,S,stride,takes", [
    (3, 112, 112, 32, 64, 3, 3, 1, True), (5, 224, 224, 10, 32, 3, 3, 1, True), (8, 56, 56, 80, 64, 3, 3, 1, True),
    (4, 112, 112, 17, 64, 3, 3, 1, False), (4, 28, 69, 412, 64, 3, 3, 2, False), (3, 14, 14, 686, 16, 3, 3, 1, False),
    (8, 28, 28, 213, 32, 1, 3, 1, False), (8, 56, 56, 49, 64, 3, 3, 1, False), (9, 56, 56, 52, 64, 3, 3, 1, True)])
def test_short_reductions_take_the_kernel_where_it_pays(P, C, H, W, N, K, R, S, stride, takes):
    import torch
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("sizes for 256 compute units")
    x, w = torch.randn(N, C, H, W, device="cuda"), torch.randn(K, C, R, S, device="cuda")
    P.conv2d_fwd(x, w, stride=stride, pad=1)
    assert (P.get_last_tile().algo == 3) == takes


# more than two units a wave: in runs of neighbours (rows read again) and in steps over the card, with and without some left over
@pytest.mark.parametrize("s", [synth.ConvShape("runs", 6, 3, 224, 221, 8, 3, 3, 1, 1), synth.ConvShape("runs_none_left", 8, 2, 256, 128, 5, 5, 5, 1, 2),
                               synth.ConvShape("steps", 1601, 4, 14, 15, 9, 3, 3, 1, 1), synth.ConvShape("steps_none_left", 2048, 3, 16, 16, 6, 3, 3, 2, 1),
                               synth.ConvShape("steps_strided", 23, 3, 223, 227, 7, 3, 3, 2, 1)], ids=lambda s: s.name)
def test_units_of_a_wave(P, s):
    x, w, b = synth.conv_inputs(s, seed=7, dist="normal", bias=True)
    want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad)
    P.set_tile_override(P.TileCfg(**THIN))
    got = host(P.conv2d_fwd(dev(x), dev(w), dev(b), stride=s.stride, pad=s.pad))
    P.set_tile_override(None)
    assert oracle.scaled_error(got, want, ab) <= FP32_TOL


# fewer pixels than a unit, fewer units than waves, one channel in and out, a filter larger than the image, 63 and 1 taps
FORCED = [synth.ConvShape("one_pixel", 1, 5, 3, 3, 7, 3, 3, 1, 0), synth.ConvShape("one_unit", 1, 1, 8, 8, 1, 1, 1, 1, 0),
          synth.ConvShape("units_65", 3, 7, 37, 37, 64, 5, 5, 1, 2), synth.ConvShape("large_filter", 2, 6, 5, 4, 33, 9, 7, 1, 4),
          synth.ConvShape("strided_past_the_end", 2, 42, 11, 13, 64, 3, 3, 4, 1), synth.ConvShape("1x1_384", 3, 384, 9, 7, 64, 1, 1, 1, 0)]


@pytest.mark.parametrize("s", FORCED + SHAPES, ids=lambda s: s.name)
def test_forced_on_any_problem_it_fits(P, s):
    x, w, b = synth.conv_inputs(s, seed=5, dist="normal", bias=True)
    want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad, act="relu")
    P.set_tile_override(P.TileCfg(**THIN))
    got = host(P.conv2d_fwd(dev(x), dev(w), dev(b), stride=s.stride, pad=s.pad, act="relu"))
    P.set_tile_override(None)
    assert oracle.scaled_error(got, want, ab) <= FP32_TOL


def test_forced_on_a_problem_it_does_not_fit(P):
    for s in (synth.ConvShape("65_channels", 1, 3, 9, 9, 65, 3, 3, 1, 1), synth.ConvShape("64_taps", 1, 3, 9, 9, 8, 8, 8, 1, 4),
              synth.ConvShape("387_rows", 1, 43, 9, 9, 8, 3, 3, 1, 1)):
        x, w, _ = synth.conv_inputs(s, seed=6, dist="normal")
        P.set_tile_override(P.TileCfg(**THIN))
        with pytest.raises(P.PolydlError):
            P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad)
        P.set_tile_override(None)


def test_through_every_entry_captured_and_misaligned(P):
    import torch
    s = SHAPES[0]
    x, w, b = synth.conv_inputs(s, seed=8, dist="normal", bias=True)
    want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad, act="relu")
    kw = dict(stride=s.stride, pad=s.pad, act="relu")
    dx, dw, db = dev(x), dev(w), dev(b)
    eager = P.conv2d_fwd(dx, dw, db, **kw)
    assert oracle.scaled_error(host(eager), want, ab) <= FP32_TOL

    def ran(out):
        assert P.get_last_tile().as_dict() == THIN
        assert torch.equal(out, eager)

    ran(P.conv2d_fwd(dx, dw, db, w_tap=P.filter_tap_copy(dw), **kw))
    ran(P.conv2d_fwd_noalloc(dx, dw, db, torch.full_like(eager, -1.0), **kw))

    def off_by_one(t):       # four bytes past the allocation's alignment
        v = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
        return v.copy_(t)

    ran(P.conv2d_fwd(off_by_one(dx), off_by_one(dw), off_by_one(db), out=off_by_one(eager).fill_(-1.0), **kw))

    out = torch.empty_like(eager)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        P.conv2d_fwd(dx, dw, db, out=out, **kw)
    for rep in range(4):
        out.fill_(-1.0)
        graph.replay()
        torch.cuda.synchronize()
        ran(out)
        P.conv2d_fwd(dx, dw, db, **kw)       # eager work between the replays


@pytest.mark.parametrize("C", [3, 4], ids=["filter_rows_of_75", "filter_rows_of_100"])   # dword and 128-bit filter loads
def test_short_reduction_on_every_tile(P, C):
    # every fp32 gather variant on a grid of several rounds: whole tiles, cut leftover tiles, two parts; every output compared
    import torch
    s = synth.ConvShape("b", 64, C, 28, 15, 512, 5, 5, 1, 2)
    x, w, b = synth.conv_inputs(s, seed=11 + C, dist="normal", bias=True)
    want, ab = (torch.from_numpy(a).cuda() for a in oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad))
    dx, dw, db = dev(x), dev(w), dev(b)
    for v in P.variants(0):
        if v.algo != 0:
            continue
        for v.split_k, v.raster in ((1, 1), (1, 3), (2, 1)):
            P.set_tile_override(v)
            first = P.conv2d_fwd(dx, dw, db, stride=s.stride, pad=s.pad)
            assert bool(((first.double() - want).abs() <= FP32_TOL * ab).all()), v
            assert torch.equal(first, P.conv2d_fwd(dx, dw, db, stride=s.stride, pad=s.pad)), v
    P.set_tile_override(None)


# two steps, the most steps, an odd number of pairs; 98304 pixels and a few
REDO = [synth.ConvShape("two_steps", 1, 3, 320, 321, 64, 3, 3, 1, 1), synth.ConvShape("24_steps", 1, 6, 318, 331, 33, 7, 9, 1, 4),
        synth.ConvShape("six_steps", 9, 9, 105, 105, 40, 3, 3, 1, 1)]


@pytest.mark.parametrize("where", ["first_block", "second_block", "both_blocks", "filter_tiny", "filter_rounds_to_inf"])
@pytest.mark.parametrize("s", REDO, ids=lambda s: s.name)
def test_recomputed_pixel_blocks(P, s, where):
    # which of a unit's two blocks of 32 pixels is recomputed, and from which copy of the filter; the rest of the unit stays
    x, w, b = synth.conv_inputs(s, seed=21, dist="normal", bias=True)
    before = None
    if where == "filter_rounds_to_inf":
        x *= np.float32(1e-3)
        w[3, 1, 0, 0] = np.finfo(np.float32).max    # its first part is an infinity
    elif where == "filter_tiny":
        w[s.K - 1] *= np.float32(1e-36)
        w[0] *= np.float32(2.0 ** 40)
    else:
        before = host(P.conv2d_fwd(dev(x), dev(w), dev(b), stride=s.stride, pad=s.pad, pre_act="relu6"))
        # one pixel per recomputed block, far from the others' taps; stride 1 and padding: outputs lie where the inputs do
        for q in {"first_block": [8], "second_block": [40], "both_blocks": [8, 55]}[where]:
            r, c = divmod((s.H // 2 * s.W // 64) * 64 + q, s.W)
            x[0, :, r, c] = np.float32(1.17e-38) * np.float32(1.3)
    want, ab = oracle.conv2d_fwd(np.clip(x, 0, 6), w, bias=b, stride=s.stride, pad=s.pad)
    got = host(P.conv2d_fwd(dev(x), dev(w), dev(b), stride=s.stride, pad=s.pad, pre_act="relu6"))
    # one rounding per product and addition of a sequential sum bounds either instruction
    assert (np.abs(got - want) <= (s.C * s.R * s.S + 2) * 2.0 ** -24 * ab).all()
    if before is not None:
        far = np.ones(got.shape, bool)
        for q in (8, 40, 55):
            r, c = divmod((s.H // 2 * s.W // 64) * 64 + q, s.W)
            far[0, :, max(0, r - s.R):r + s.R + 1] = False
        assert np.array_equal(got[far], before[far])
