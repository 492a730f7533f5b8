"""Small problems on single waves (a tile of 64x64 or 32x32 whose reduction the eight waves of a workgroup share): edges of tiles,
steps and parts, tap masks, values the split cannot hold, and the calls that go there, against the oracle."""
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
    p.set_tile_override(None)


def wave(P, tile, parts, layout=0, waves=8):
    return P.TileCfg(tile, tile, 16, tile, tile, parts, layout, 1 if waves == 8 else 0, 0, 0)


TILES = [(64, 8), (64, 4), (32, 8)]       # tile and the waves that share it


# rows and columns at, one below and one past the tiles, reductions at, below and past steps, waves and parts; one row, one column
@pytest.mark.parametrize("tile,waves", TILES)
@pytest.mark.parametrize("M,N,K", [(64, 64, 128), (63, 65, 127), (65, 31, 129), (1, 33, 16), (33, 1, 15), (130, 97, 3), (31, 200, 700),
                                   (600, 95, 1000), (5, 3, 4100)])
def test_sgemm(P, tile, waves, M, N, K):
    import torch
    A, B, C0 = synth.sgemm_inputs(M, N, K, seed=M + N, c0="random")
    want, ab = oracle.gemm(A, B, C0)
    ints = synth.sgemm_inputs(M, N, K, seed=K, dist="ints")
    for parts in (1, 2, 5):
        P.set_tile_override(wave(P, tile, parts, waves=waves))
        got = host(P.sgemm(dev(A), dev(B), dev(C0)))
        assert oracle.scaled_error(got, want, ab) <= FP32_TOL, parts
        out = torch.full((M, N), float("nan"), device="cuda")
        got = host(P.sgemm(dev(ints[0]), dev(ints[1]), out, alpha=1.0, beta=0.0))
        assert np.array_equal(got.astype(np.float64), ints[0].astype(np.float64) @ ints[1].astype(np.float64)), parts
    P.set_tile_override(None)


SHAPES = [synth.ConvShape("3x3", 2, 16, 9, 11, 70, 3, 3, 1, 1), synth.ConvShape("ragged", 3, 21, 13, 7, 33, 3, 3, 2, 1),
          synth.ConvShape("tap_steps", 2, 48, 10, 9, 65, 3, 3, 1, 1), synth.ConvShape("small_images", 40, 32, 3, 3, 31, 3, 3, 1, 1),
          synth.ConvShape("31_taps", 1, 10, 6, 40, 20, 1, 31, 1, 15), synth.ConvShape("32_taps", 1, 16, 12, 13, 40, 4, 8, 1, 3),
          synth.ConvShape("63_taps", 1, 6, 18, 31, 33, 7, 9, 1, 4), synth.ConvShape("strided_5x5", 2, 32, 17, 15, 70, 5, 5, 3, 2),
          synth.ConvShape("no_padding", 1, 5, 8, 8, 64, 2, 2, 2, 0), synth.ConvShape("past_the_image", 2, 7, 5, 4, 9, 9, 7, 1, 4),
          synth.ConvShape("1x1", 3, 67, 9, 7, 100, 1, 1, 1, 0), synth.ConvShape("1x1_strided", 2, 130, 8, 9, 33, 1, 1, 2, 0),
          synth.ConvShape("1x1_padded", 2, 20, 6, 5, 10, 1, 1, 1, 1), synth.ConvShape("one_of_each", 1, 1, 1, 1, 1, 1, 1, 1, 0),
          synth.ConvShape("many_parts", 1, 256, 4, 4, 40, 3, 3, 1, 1)]


@pytest.mark.parametrize("s", SHAPES, ids=lambda s: s.name)
def test_conv(P, s):
    x, w, b = synth.conv_inputs(s, seed=11 + s.C, dist="normal", bias=True)
    xi, wi, bi = synth.conv_inputs(s, seed=12 + s.C, dist="ints", bias=True)
    dx, dw, db = dev(x), dev(w), dev(b)
    tap = dict(w_tap=P.filter_tap_copy(dw))
    applies = 2 <= s.R * s.S <= 63 and s.C % 16 == 0
    exact, _ = oracle.conv2d_fwd(xi, wi, bias=bi, stride=s.stride, pad=s.pad)
    for act, bias, pre, kw in (("relu6", True, None, {}), ("none", False, "relu", {}), ("relu", True, None, tap)):
        layout = 2 if kw and applies else 0
        want, ab = oracle.conv2d_fwd(np.maximum(x, 0) if pre else x, w, bias=b if bias else None, stride=s.stride, pad=s.pad, act=act)
        for tile, waves in TILES:
            for parts in (1, 3):
                P.set_tile_override(wave(P, tile, parts, layout, waves))
                got = host(P.conv2d_fwd(dx, dw, db if bias else None, stride=s.stride, pad=s.pad, act=act, pre_act=pre, **kw))
                assert P.get_last_tile().wm == tile
                assert oracle.scaled_error(got, want, ab) <= FP32_TOL, (tile, parts, act)
                if act == "relu6":
                    got = host(P.conv2d_fwd(dev(xi), dev(wi), dev(bi), stride=s.stride, pad=s.pad))
                    assert np.array_equal(got.astype(np.float64), exact), (tile, parts)
    P.set_tile_override(None)


def test_refused(P):
    for s, layout in ((synth.ConvShape("64_taps", 1, 3, 9, 9, 8, 8, 8, 1, 4), 0), (synth.ConvShape("no_copy", 1, 16, 9, 9, 8, 3, 3, 1, 1), 2)):
        x, w, _ = synth.conv_inputs(s, seed=6, dist="normal")
        P.set_tile_override(wave(P, 32, 1, layout))
        with pytest.raises(P.PolydlError) as err:
            P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad)
        assert err.value.status == -3
    P.set_tile_override(None)
    for bad in (P.TileCfg(64, 64, 16, 64, 64, 1, 0, 2, 0, 0), P.TileCfg(32, 32, 16, 32, 32, 1, 0, 0, 0, 0), P.TileCfg(32, 64, 16, 32, 64, 1, 0, 1, 0, 0)):
        with pytest.raises(P.PolydlError):
            P.set_tile_override(bad)


# Values the split cannot hold: in the tile, and behind a row's end, where a ragged reduction reads the next row's first values
@pytest.mark.parametrize("tile,waves", TILES)
@pytest.mark.parametrize("case", ["inf", "nan", "largest", "tiny", "row_ends"])
def test_values_the_split_cannot_hold(P, tile, waves, case):
    M, N, K = 70, 75, 333
    r = np.random.default_rng(5)
    A, B = r.uniform(-1, 1, (M, K)).astype(np.float32), r.uniform(-1, 1, (K, N)).astype(np.float32)
    if case == "inf":
        A[3, 332] = np.inf
    elif case == "nan":
        B[0, 74] = np.nan
    elif case == "largest":
        A[69, 5] = np.finfo(np.float32).max
        B[5] *= np.float32(1e-3)
    elif case == "tiny":
        A[:, 100:] *= np.float32(1e-37)
        B[100:] *= np.float32(1e20)
    else:                       # row 41 of A and row 0 of B begin with infinities, which no other row may see
        A[41, :5] = -np.inf
        B[0, :9] = np.inf
    C0 = np.zeros((M, N), np.float32)
    with np.errstate(all="ignore"):
        want = A.astype(np.float64) @ B.astype(np.float64)
        ab = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    for parts in (1, 2):
        P.set_tile_override(wave(P, tile, parts, waves=waves))
        got = host(P.sgemm(dev(A), dev(B), dev(C0)))
        ok = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        assert np.array_equal(got[np.isinf(want)], want[np.isinf(want)].astype(np.float32))
        assert (np.abs(got[ok] - want[ok]) <= FP32_TOL * ab[ok]).all(), parts
    P.set_tile_override(None)


@pytest.mark.parametrize("case", ["inf", "tiny", "tiny_filter"])
def test_conv_values_the_split_cannot_hold(P, case):
    for s in (synth.ConvShape("ragged", 2, 21, 9, 8, 40, 3, 3, 1, 1), synth.ConvShape("1x1", 2, 37, 6, 7, 70, 1, 1, 1, 0)):
        x, w, _ = synth.conv_inputs(s, seed=9, dist="normal")
        if case == "inf":
            x[1, 3, 4, 5] = np.inf
            if s.pad == 0:
                w[5, 0, 0, 0] = -np.inf      # the value behind the end of row 4
        elif case == "tiny":
            x[:, 5:] *= np.float32(1e-37)
            w *= np.float32(1e20)
        else:
            w[:, 7:] *= np.float32(1e-37)
        with np.errstate(all="ignore"):
            want, ab = oracle.conv2d_fwd(x, w, stride=s.stride, pad=s.pad)
        ok = np.isfinite(want)
        for tile in (64, 32):
            P.set_tile_override(wave(P, tile, 2))
            got = host(P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad))
            assert np.array_equal(np.isfinite(got), ok)
            assert (np.abs(got[ok] - want[ok]) <= FP32_TOL * ab[ok] + 1e-44).all(), (s.name, tile)
    P.set_tile_override(None)


@pytest.mark.parametrize("case", ["inf", "tiny", "tiny_filter"])
def test_conv_values_the_split_cannot_hold_on_four_waves_and_tap_by_tap(P, case):
    s = synth.ConvShape("copy", 2, 48, 9, 8, 70, 3, 3, 1, 1)
    x, w, b = synth.conv_inputs(s, seed=23, dist="normal", bias=True)
    if case == "inf":
        x[1, 3, 4, 5] = np.inf
    elif case == "tiny":
        x[:, 5:] *= np.float32(1e-37)
        w *= np.float32(1e20)
    else:
        w[:, 7:] *= np.float32(1e-37)
    dx, dw, db = dev(x), dev(w), dev(b)
    tap = P.filter_tap_copy(dw)
    with np.errstate(all="ignore"):
        want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad)
    ok = np.isfinite(want)
    for tile, waves in TILES:
        for layout, kw in ((0, {}), (2, dict(w_tap=tap))):
            for parts in (1, 3):
                P.set_tile_override(wave(P, tile, parts, layout, waves))
                got = host(P.conv2d_fwd(dx, dw, db, stride=s.stride, pad=s.pad, **kw))
                assert np.array_equal(np.isfinite(got), ok), (tile, waves, layout, parts)
                assert (np.abs(got[ok] - want[ok]) <= FP32_TOL * ab[ok] + 1e-44).all(), (tile, waves, layout, parts)
    P.set_tile_override(None)


def test_the_library_goes_there(P):
    import torch
    # by itself for small problems, aligned or not, and through the entry with the fixed scratch memory; not for large ones, one-step ones
    s = synth.ConvShape("small", 1, 64, 56, 56, 64, 3, 3, 1, 1)
    x, w, b = synth.conv_inputs(s, seed=13, dist="normal", bias=True)
    want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad, act="relu")
    kw = dict(stride=s.stride, pad=s.pad, act="relu")
    dx, dw, db = dev(x), dev(w), dev(b)
    eager = P.conv2d_fwd(dx, dw, db, **kw)
    tile = P.get_last_tile()
    assert tile.wm == tile.bm and tile.bm in (32, 64) and tile.algo == 0
    assert oracle.scaled_error(host(eager), want, ab) <= FP32_TOL
    assert P.model_conv2d(tuple(s)[1:], tile).predicted_us > 0

    def skew(t):       # four bytes past the allocation's alignment
        v = torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape)
        return v.copy_(t)

    for out in (P.conv2d_fwd(skew(dx), skew(dw), skew(db), out=skew(eager).fill_(-1.0), **kw),
                P.conv2d_fwd_noalloc(dx, dw, db, torch.full_like(eager, -1.0), **kw)):
        assert P.get_last_tile().as_dict() == tile.as_dict()
        assert torch.equal(out, eager)
    A, B, _ = synth.sgemm_inputs(500, 520, 510, seed=3)
    C = torch.zeros(500, 520, device="cuda")
    P.sgemm(dev(A), dev(B), C)
    small = P.get_last_tile()
    assert small.wm == small.bm
    assert P.model_sgemm(500, 520, 510, small).predicted_us > 0
    big = torch.zeros(4096, 4096, device="cuda")
    P.sgemm(big, big, big.clone())
    assert P.get_last_tile().bm > 64
    thin = torch.zeros(500, 16, device="cuda")
    P.sgemm(thin, thin.view(16, 500), torch.zeros(500, 500, device="cuda"))
    last = P.get_last_tile()
    assert last.wm < last.bm
    P.conv2d_fwd(torch.zeros(1, 16, 20, 20, device="cuda"), torch.zeros(64, 16, 1, 1, device="cuda"))
    last = P.get_last_tile()
    assert not (last.algo == 0 and last.wm == last.bm)


# parts that meet in the library's fixed array: forced ones of every tile, the larger problem first, and a choice of the library's own
@pytest.mark.parametrize("captured", [False, True])
def test_several_parts_on_the_fixed_scratch_memory(P, captured):
    import torch
    forced = [wave(P, tile, parts, waves=waves) for tile, waves in TILES for parts in (3, 5)]
    for s, tiles in ((synth.ConvShape("a", 3, 48, 13, 11, 150, 3, 3, 1, 1), forced), (synth.ConvShape("b", 1, 32, 6, 6, 20, 3, 3, 2, 1), forced),
                     (synth.ConvShape("long", 1, 512, 14, 14, 256, 3, 3, 1, 1), [None])):
        x, w, b = synth.conv_inputs(s, seed=22, dist="normal", bias=True)
        dx, dw, db = dev(x), dev(w), dev(b)
        kw = dict(stride=s.stride, pad=s.pad, act="relu")
        want, ab = oracle.conv2d_fwd(x, w, bias=b, stride=s.stride, pad=s.pad, act="relu")
        for tile in tiles:
            P.set_tile_override(tile)
            ref = host(P.conv2d_fwd(dx, dw, db, **kw))
            last = P.get_last_tile()
            assert last.split_k > 1 and last.wm == last.bm and last.algo == 0, last
            assert oracle.scaled_error(ref, want, ab) <= FP32_TOL, (s.name, last)
            out = torch.full(ref.shape, -1.0, device="cuda")

            def call():
                P.conv2d_fwd_noalloc(dx, dw, db, out, **kw)
            if captured:
                side = torch.cuda.Stream()
                graph = torch.cuda.CUDAGraph()
                torch.cuda.synchronize()
                with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
                    call()
            for _ in range(3 if captured else 1):
                out.fill_(-1.0)
                torch.cuda.synchronize()
                graph.replay() if captured else call()
                assert P.get_last_tile().as_dict() == last.as_dict()
                assert np.array_equal(host(out), ref), (s.name, last)
                if captured:        # eager work in between, on the same array
                    call()
                    torch.cuda.synchronize()
    P.set_tile_override(None)


def test_short_reductions_stay_as_exact(P):
    # what the library does by itself is no further from 64 bits than its ranked pick (0.5 %: single sums differ in either direction)
    import torch

    def off(got, want):
        return np.linalg.norm(host(got) - want) / np.linalg.norm(want)

    for M, N, K in ((411, 1388, 32), (411, 1388, 40), (300, 500, 72), (1000, 64, 96), (300, 500, 112), (64, 64, 128), (411, 1388, 200)):
        A, B, _ = synth.sgemm_inputs(M, N, K, seed=M + K)
        want = A.astype(np.float64) @ B.astype(np.float64)
        C = torch.zeros(M, N, device="cuda")
        here = off(P.sgemm(dev(A), dev(B), C, alpha=1.0, beta=0.0), want)
        P.set_tile_override(P.pick_sgemm(M, N, K)[0])
        assert here <= 1.005 * off(P.sgemm(dev(A), dev(B), C, alpha=1.0, beta=0.0), want), (M, N, K)
        P.set_tile_override(None)
    for s in (synth.ConvShape("144", 1, 16, 7, 7, 64, 3, 3, 2, 1), synth.ConvShape("128", 2, 128, 14, 14, 128, 1, 1, 1, 0)):
        x, w, _ = synth.conv_inputs(s, seed=21, dist="normal")
        want, _ = oracle.conv2d_fwd(x, w, stride=s.stride, pad=s.pad)
        here = off(P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad), want)
        P.set_tile_override(P.pick_conv2d(tuple(s)[1:])[0])
        assert here <= 1.005 * off(P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad), want), s.name
        P.set_tile_override(None)


BF16 = SHAPES + [synth.ConvShape("two_steps", 2, 64, 5, 7, 40, 1, 1, 1, 0), synth.ConvShape("41_steps", 1, 144, 9, 9, 70, 3, 3, 1, 1)]


@pytest.mark.parametrize("s", BF16, ids=lambda s: s.name)
def test_bf16(P, s):
    import torch
    x, w, b = synth.conv_inputs(s, seed=14 + s.C, dist="normal", bias=True)
    xi, wi, bi = synth.conv_inputs(s, seed=15 + s.C, dist="ints", bias=True)
    exact, _ = oracle.conv2d_fwd(xi, wi, bias=bi, stride=s.stride, pad=s.pad)
    tx, tw = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, w))
    want, ab = oracle.conv2d_fwd(host(tx.float()), host(tw.float()), bias=b, stride=s.stride, pad=s.pad, act="relu")
    blocked = lambda a, f: (P.nchw_to_nchwc_bf16(a, 8), P.kcrs_to_kcrsck_bf16(f, 8, 1))
    for tile, waves in TILES:
        for parts in (1, 2, 5):
            P.set_tile_override(wave(P, tile, parts, waves=waves))
            got = host(P.conv2d_fwd_bf16_blocked(*blocked(tx, tw), s.C, dev(b), stride=s.stride, pad=s.pad, act="relu"))
            assert oracle.scaled_error(got, want, ab) <= FP32_TOL, (tile, parts)      # products of bfloat16 values are exact in fp32
            ints = [torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (xi, wi)]
            got = host(P.conv2d_fwd_bf16_blocked(*blocked(*ints), s.C, dev(bi), stride=s.stride, pad=s.pad))
            assert np.array_equal(got.astype(np.float64), exact), (tile, parts)
    P.set_tile_override(None)


def test_bf16_infinity_at_the_end_of_a_filter_row(P):
    # the reduction ends inside a step: what lies behind a row's end is the next row, which begins with an infinity
    import torch
    s = synth.ConvShape("ends", 1, 40, 6, 6, 40, 1, 1, 1, 0)
    x, w, _ = synth.conv_inputs(s, seed=16, dist="normal")
    w[5, 0] = np.inf
    for tile in (64, 32):
        P.set_tile_override(wave(P, tile, 1))
        tx, tw = (torch.from_numpy(a).cuda().to(torch.bfloat16) for a in (x, w))
        got = host(P.conv2d_fwd_bf16(tx, tw))
        assert np.isfinite(got[:, :5]).all() and np.isfinite(got[:, 6:]).all() and not np.isfinite(got[:, 5]).any()
    P.set_tile_override(None)


def test_bf16_the_library_goes_there_and_is_captured(P):
    import torch
    s = synth.ConvShape("small", 1, 512, 14, 14, 128, 3, 3, 1, 1)
    x, w, b = synth.conv_inputs(s, seed=17, dist="normal", bias=True)
    tx, tw, tb = torch.from_numpy(x).cuda().to(torch.bfloat16), torch.from_numpy(w).cuda().to(torch.bfloat16), dev(b)
    x8, w8 = P.nchw_to_nchwc_bf16(tx, 8), P.kcrs_to_kcrsck_bf16(tw, 8, 1)
    out = torch.empty(1, 128, 14, 14, device="cuda")
    call = lambda: P.conv2d_fwd_bf16_blocked(x8, w8, s.C, tb, out=out, stride=1, pad=1, act="relu")
    eager = host(call())
    tile = P.get_last_tile()
    assert tile.wm == tile.bm
    assert P.model_conv2d_bf16(tuple(s)[1:], tile) > 0
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        call()                              # its scratch memory
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            call()
    for _ in range(3):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(host(out), eager)
        call()
        torch.cuda.synchronize()


@pytest.mark.parametrize("s", [synth.ConvShape("single_waves", 1, 512, 14, 14, 128, 3, 3, 1, 1),
                               synth.ConvShape("ranked_64_taps", 1, 256, 12, 12, 64, 8, 8, 1, 3)], ids=lambda s: s.name)
def test_bf16_is_captured_without_scratch_memory(P, s):
    # a choice that splits its reduction when called eagerly, on a stream that has no scratch memory: the capture records the best
    # choice that needs none
    import torch
    x, w, b = synth.conv_inputs(s, seed=18, dist="normal", bias=True)
    tx, tw, tb = torch.from_numpy(x).cuda().to(torch.bfloat16), torch.from_numpy(w).cuda().to(torch.bfloat16), dev(b)
    want, ab = oracle.conv2d_fwd(host(tx.float()), host(tw.float()), bias=b, stride=s.stride, pad=s.pad, act="relu")
    x8, w8 = P.nchw_to_nchwc_bf16(tx, 8), P.kcrs_to_kcrsck_bf16(tw, 8, 1)
    out = torch.empty(want.shape, dtype=torch.float32, device="cuda")

    def call():
        P.conv2d_fwd_bf16_blocked(x8, w8, s.C, tb, out=out, stride=s.stride, pad=s.pad, act="relu")
    call()                                  # on the default stream: it has its own scratch memory
    torch.cuda.synchronize()
    eager = P.get_last_tile()
    assert eager.split_k > 1, eager
    fresh = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(fresh):
        with torch.cuda.graph(graph, stream=fresh):
            call()
            captured = P.get_last_tile()
    assert captured.split_k == 1, captured
    for _ in range(3):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert oracle.scaled_error(host(out), want, ab) <= FP32_TOL
        call()                              # eager work in between
        torch.cuda.synchronize()
        assert P.get_last_tile().as_dict() == eager.as_dict()      # the choice for eager calls is unchanged
        assert oracle.scaled_error(host(out), want, ab) <= FP32_TOL


# layers that the single waves made slower than their ranked pick (percent more time), which therefore stay with it
SLOWER = [synth.ConvShape("few_channels_strided_29", 32, 128, 56, 45, 64, 1, 1, 2, 0), synth.ConvShape("few_channels_17", 64, 128, 7, 39, 64, 1, 1, 1, 0),
          synth.ConvShape("few_channels_strided_25", 32, 256, 19, 104, 64, 1, 1, 2, 0), synth.ConvShape("few_channels_long_8", 32, 512, 28, 86, 64, 1, 1, 2, 0),
          synth.ConvShape("strided_10", 32, 128, 28, 28, 128, 1, 1, 2, 0), synth.ConvShape("strided_12", 33, 128, 72, 26, 128, 1, 1, 2, 0),
          synth.ConvShape("stride_3_26", 53, 128, 68, 68, 128, 1, 1, 3, 0),
          synth.ConvShape("large_strided_17", 35, 1024, 28, 96, 128, 1, 1, 2, 0), synth.ConvShape("large_28", 4, 2925, 135, 83, 18, 1, 1, 1, 0),
          synth.ConvShape("many_lines_30", 53, 788, 9, 9, 284, 1, 1, 3, 0),
          synth.ConvShape("large_into_few_10", 65, 1024, 17, 17, 64, 1, 1, 2, 0), synth.ConvShape("unstrided_6", 36, 128, 7, 5, 512, 1, 1, 1, 0)]


def stays(P, s, call):
    import torch
    x, w = torch.zeros(s.N, s.C, s.H, s.W, device="cuda"), torch.zeros(s.K, s.C, s.R, s.S, device="cuda")
    call(x, w)
    torch.cuda.synchronize()
    t = P.get_last_tile()
    assert not (t.algo == 0 and t.wm == t.bm), t


@pytest.mark.parametrize("s", SLOWER, ids=lambda s: s.name)
def test_1x1_layers_that_would_be_slower_stay(P, s):
    import torch
    kw = dict(stride=s.stride, pad=s.pad)
    stays(P, s, lambda x, w: P.conv2d_fwd(x, w, **kw))
    stays(P, s, lambda x, w: P.conv2d_fwd_noalloc(x, w, None, torch.empty((s.N, s.K) + tuple(synth.out_hw(s)), device="cuda"), **kw))


# loads over many cache lines, outputs far smaller than their input; percent more time in the KCRS order, with the filter's copy
@pytest.mark.parametrize("s", [synth.ConvShape("37_58", 85, 688, 4, 4, 1438, 4, 3, 1, 0), synth.ConvShape("17_15", 95, 512, 7, 7, 512, 3, 3, 3, 0),
                               synth.ConvShape("32_31", 103, 512, 7, 7, 128, 4, 4, 2, 0), synth.ConvShape("21_21", 101, 128, 7, 7, 256, 4, 4, 2, 0)],
                         ids=lambda s: s.name)
def test_scattered_layers_that_would_be_slower_stay(P, s):
    import torch
    kw = dict(stride=s.stride, pad=s.pad)
    stays(P, s, lambda x, w: P.conv2d_fwd(x, w, **kw))
    stays(P, s, lambda x, w: P.conv2d_fwd(x, w, w_tap=P.filter_tap_copy(w), **kw))
    stays(P, s, lambda x, w: P.conv2d_fwd_noalloc(x, w, None, torch.empty((s.N, s.K) + tuple(synth.out_hw(s)), device="cuda"), **kw))


@pytest.mark.parametrize("s", [synth.ConvShape("3x3_9", 32, 1019, 28, 28, 64, 3, 3, 1, 1), synth.ConvShape("5x5_8", 32, 256, 56, 14, 64, 5, 5, 1, 2),
                               synth.ConvShape("7x7_leftover_10", 32, 39, 87, 63, 35, 7, 7, 1, 3)], ids=lambda s: s.name)
def test_layers_of_few_channels_that_would_be_slower_stay(P, s):
    stays(P, s, lambda x, w: P.conv2d_fwd(x, w, stride=s.stride, pad=s.pad))


@pytest.mark.parametrize("s", [synth.ConvShape("few_channels_29", 64, 512, 56, 20, 64, 3, 3, 2, 1), synth.ConvShape("few_channels_7x7_91", 64, 512, 14, 18, 64, 7, 7, 2, 3),
                               synth.ConvShape("few_channels_one_part_12", 32, 512, 47, 47, 32, 3, 3, 2, 1),
                               synth.ConvShape("many_channels_12", 32, 256, 28, 16, 256, 3, 3, 2, 1),
                               synth.ConvShape("large_66", 17, 3856, 51, 9, 102, 5, 5, 2, 0), synth.ConvShape("large_186", 74, 3264, 21, 9, 23, 4, 4, 2, 0)],
                         ids=lambda s: s.name)
def test_strided_layers_with_the_filter_copy_that_would_be_slower_stay(P, s):
    stays(P, s, lambda x, w: P.conv2d_fwd(x, w, stride=s.stride, pad=s.pad, w_tap=P.filter_tap_copy(w)))


@pytest.mark.parametrize("s", [synth.ConvShape("strided_26", 36, 803, 28, 28, 256, 3, 3, 2, 1), synth.ConvShape("strided_short_13", 64, 128, 56, 56, 64, 3, 3, 2, 1),
                               synth.ConvShape("few_channels_17", 14, 128, 56, 56, 17, 3, 3, 1, 1), synth.ConvShape("few_steps_13", 64, 16, 14, 23, 29, 3, 3, 1, 1),
                               synth.ConvShape("five_steps_20", 49, 10, 8, 43, 2, 3, 3, 1, 1), synth.ConvShape("three_steps_16", 12, 5, 63, 26, 2, 3, 3, 1, 1),
                               synth.ConvShape("large_70", 28, 1669, 30, 110, 28, 3, 3, 1, 1), synth.ConvShape("1x1_22", 109, 2352, 17, 20, 68, 1, 1, 1, 0),
                               synth.ConvShape("large_filter_87", 18, 2513, 100, 3, 743, 3, 3, 3, 0), synth.ConvShape("large_filter_75", 19, 3217, 100, 3, 367, 3, 3, 3, 0),
                               synth.ConvShape("1x1_strided_30", 105, 94, 173, 19, 34, 1, 1, 3, 0), synth.ConvShape("1x1_long_24", 58, 3077, 34, 18, 176, 1, 1, 1, 0),
                               synth.ConvShape("three_steps_10", 3, 7, 32, 32, 142, 3, 3, 1, 1), synth.ConvShape("three_steps_11", 126, 1, 20, 2, 64, 3, 3, 1, 1)],
                         ids=lambda s: s.name)
def test_bf16_layers_that_would_be_slower_stay(P, s):
    import torch
    stays(P, s, lambda x, w: P.conv2d_fwd_bf16(x.to(torch.bfloat16), w.to(torch.bfloat16), stride=s.stride, pad=s.pad))


@pytest.mark.parametrize("M,N,K", [(105, 236, 466615), (326, 58, 380505), (256, 64, 400000), (69, 59, 388422)])
def test_long_products_that_would_be_slower_stay(P, M, N, K):
    import torch
    P.sgemm(torch.zeros(M, K, device="cuda"), torch.zeros(K, N, device="cuda"), torch.zeros(M, N, device="cuda"))
    torch.cuda.synchronize()
    t = P.get_last_tile()
    assert t.wm < t.bm, t
