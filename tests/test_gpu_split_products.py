"""Products formed on the bfloat16 matrix cores from three-way split operands: error against 64 bits, and
values the split cannot hold (infinities, NaN, the largest and the smallest numbers), which the kernels
recompute in fp32."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2006_02230_amd as p
    yield p
    p.set_tile_override(None)


def split_tiles(P):
    return [v for v in P.variants(1) if v.bk == 16 and v.wm * v.wn <= 64 * 64]


# one stage, its boundary, the boundaries of the unrolled pipeline, long
@pytest.mark.parametrize("K", [1, 15, 16, 17, 33, 48, 64, 79, 80, 81, 97, 576, 2500])
def test_sgemm_error_against_64_bits(P, K):
    # The six products kept leave out 2^-24 of a product at worst; the main accumulator rounds once per eight
    # terms (<= 2^-24 of the running sum), at the end the two accumulators are added (once more), and the small
    # one holds at most 2^-7 of the terms, so its own roundings stay below half of one of these: in all
    # (1 + K/8 + 1 + 1/2) * 2^-24, and the last part of a block of eight.  fp32 in sequence would be
    # allowed K * 2^-24.
    for v in split_tiles(P):
        for M, N in ((v.bm, v.bn), (v.bm + 1, v.bn - 1)):
            A, B, _ = synth.sgemm_inputs(M, N, K, seed=K)
            C = dev(np.zeros((M, N), np.float32))
            P.set_tile_override(v)
            P.sgemm(dev(A), dev(B), C)
            want = A.astype(np.float64) @ B.astype(np.float64)
            terms = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
            bound = (2.0 ** -25 + (K / 8 + 3) * 2.0 ** -24) * terms
            assert (np.abs(host(C) - want) <= bound).all(), (v, K)
    P.set_tile_override(None)


def special(case, M, N, K):
    A, B, _ = synth.sgemm_inputs(M, N, K, seed=7)
    if case == "inf":
        A[1, K // 2] = np.inf                       # meets planes 1, 2 of exactly representable values too
        B[:, 3] = 0.5
    elif case == "nan":
        B[K - 1, N - 2] = np.nan
    elif case == "lowest":
        A[2, :] = 0
        A[2, 0] = np.finfo(np.float32).min          # rounds to a bfloat16 infinity
        B[0, :] = 1.0
    elif case == "tiny_row":
        A[M - 1] *= np.float32(1e-36)
        A[0] = 0
        B *= np.float32(1e20)
    elif case == "tiny_column":
        B[:, 5] *= np.float32(1e-37)
        A *= np.float32(1e20)
    elif case == "subnormal":
        A[:, :] = (A * np.float32(1e-30)) * np.float32(1e-11)
        B *= np.float32(1e30)
    return A, B


@pytest.mark.parametrize("split_k", [1, 2])
@pytest.mark.parametrize("case", ["inf", "nan", "lowest", "tiny_row", "tiny_column", "subnormal"])
def test_sgemm_values_the_split_cannot_hold(P, case, split_k):
    M, N, K = 130, 140, 150
    A, B = special(case, M, N, K)
    with np.errstate(all="ignore"):
        want = A.astype(np.float64) @ B.astype(np.float64)
        terms = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    for v in split_tiles(P):
        v.split_k = split_k
        C = dev(np.zeros((M, N), np.float32))
        P.set_tile_override(v)
        P.sgemm(dev(A), dev(B), C)
        got = host(C)
        fin = np.isfinite(want)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fin], want[~fin].astype(np.float32),
                                                                                equal_nan=True), v
        # K sequential fp32 roundings at most (the recomputation's own order)
        assert (np.abs(got[fin] - want[fin]) <= (K + 2) * 2.0 ** -24 * terms[fin]).all(), v
    P.set_tile_override(None)


def conv64(x, w, stride, pad):
    """Plain fp64 convolution and the sum of the terms' magnitudes."""
    N, C, H, W = x.shape
    K, _, R, S = w.shape
    Ph, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - S) // stride + 1
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (pad, pad), (pad, pad)))
    out, ab = np.zeros((N, K, Ph, Q)), np.zeros((N, K, Ph, Q))
    with np.errstate(all="ignore"):
        for r in range(R):
            for t in range(S):
                tap = xp[:, :, r:r + (Ph - 1) * stride + 1:stride, t:t + (Q - 1) * stride + 1:stride]
                f = w[:, :, r, t].astype(np.float64)
                out += np.einsum("kc,ncpq->nkpq", f, tap)
                ab += np.einsum("kc,ncpq->nkpq", np.abs(f), np.abs(tap))
    return out, ab


CONV = [synth.ConvShape("3x3", 2, 24, 9, 11, 70, 3, 3, 1, 1), synth.ConvShape("3x3c16", 3, 32, 7, 7, 130, 3, 3, 1, 1),
        synth.ConvShape("5x5s2", 1, 16, 13, 10, 33, 5, 5, 2, 2), synth.ConvShape("1x1", 2, 131, 8, 9, 65, 1, 1, 1, 0),
        synth.ConvShape("1x1s2", 1, 160, 15, 13, 65, 1, 1, 2, 0), synth.ConvShape("8x8", 1, 3, 20, 20, 40, 8, 8, 1, 0),
        synth.ConvShape("7x7", 1, 11, 18, 17, 64, 7, 7, 2, 3)]


@pytest.mark.parametrize("case", ["plain", "inf", "nan", "lowest", "tiny"])
@pytest.mark.parametrize("s", CONV, ids=lambda s: s.name)
def test_conv(P, s, case):
    x, w, _ = synth.conv_inputs(s, seed=11, dist="normal")
    if case == "inf":
        x[0, s.C // 2, 4, 5] = np.inf
    elif case == "nan":
        w[3, 1, s.R - 1, 0] = np.nan
    elif case == "lowest":
        x[0, 1, 3, 4] = np.finfo(np.float32).min
        w *= np.float32(1e-3)
    elif case == "tiny":
        w[2] *= np.float32(1e-36)
        x *= np.float32(1e20)
    want, ab = conv64(x, w, s.stride, s.pad)
    dx, dw = dev(x), dev(w)
    tap = P.filter_tap_copy(dw)
    Kg = s.C * s.R * s.S
    fin = np.isfinite(want)
    for v in P.variants(0):
        if v.algo != 0 or v.bk != 16 or v.wm * v.wn > 64 * 64:
            continue
        for split_k, raster in ((1, 0), (2, 1), (1, 3)):
            for layout in ((0, 2) if s.C % 16 == 0 and 2 <= s.R * s.S <= 63 else (0,)):
                v.split_k, v.raster, v.layout = split_k, raster, layout
                P.set_tile_override(v)
                got = host(P.conv2d_fwd(dx, dw, stride=s.stride, pad=s.pad, w_tap=tap if layout else None))
                assert np.array_equal(np.isnan(got), np.isnan(want)), v
                assert np.array_equal(got[~fin], want[~fin].astype(np.float32), equal_nan=True), v
                # as for the matrix product, or Kg sequential roundings where a tile is recomputed
                bound = (2.0 ** -25 + (Kg / 8 + 3) * 2.0 ** -24) if case == "plain" else (Kg + 2) * 2.0 ** -24
                assert (np.abs(got[fin] - want[fin]) <= bound * ab[fin]).all(), v
    P.set_tile_override(None)


@pytest.mark.parametrize("case", ["plain", "inf", "nan", "lowest", "tiny", "tiny_pixels"])
@pytest.mark.parametrize("s", [synth.ConvShape("c64", 2, 64, 9, 10, 128, 1, 1, 1, 0), synth.ConvShape("c32", 1, 32, 7, 6, 192, 1, 1, 1, 0),
                               synth.ConvShape("c16", 3, 16, 5, 4, 256, 1, 1, 1, 0)], ids=lambda s: s.name)
def test_pointwise_conv(P, s, case):
    x, w, b = synth.conv_inputs(s, seed=13, dist="normal", bias=True)
    if case == "inf":
        x[0, 3, 4, 2] = np.inf
    elif case == "nan":
        w[37, 5] = np.nan
    elif case == "lowest":
        x[0, 1, 3, 3] = np.finfo(np.float32).min
        w *= np.float32(1e-3)
    elif case == "tiny":
        w[40] *= np.float32(1e-37)
        x *= np.float32(1e20)
        b[:] = 0
    elif case == "tiny_pixels":
        x[:, :, 2] *= np.float32(1e-37)
        w *= np.float32(1e20)
        b[:] = 0
    want, ab = conv64(x, w, 1, 0)
    want += b.astype(np.float64)[None, :, None, None]
    ab += np.abs(b)[None, :, None, None]
    v = [v for v in P.variants(0) if v.algo == 2][0]
    P.set_tile_override(v)
    got = host(P.conv2d_fwd(dev(x), dev(w), dev(b), stride=1, pad=0))
    P.set_tile_override(None)
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(got[~fin], want[~fin].astype(np.float32), equal_nan=True)
    bound = (2.0 ** -25 + (s.C / 8 + 4) * 2.0 ** -24) if case == "plain" else (s.C + 3) * 2.0 ** -24
    assert (np.abs(got[fin] - want[fin]) <= bound * ab[fin]).all()


def all_magnitudes(seed, shape, lowest=-149):
    """Random signs and mantissas, exponents uniform over every float32 number from 2^lowest on, some zeros."""
    rng = np.random.default_rng(seed)
    v = np.ldexp(1 + rng.random(shape), rng.integers(lowest, 127, shape)) * rng.choice([-1.0, 1.0], shape)
    v[rng.random(shape) < 0.05] = 0
    with np.errstate(under="ignore"):
        return v.astype(np.float32)


# One value of ordinary size beside values whose third bfloat16 part lies below the smallest bfloat16 (2^-133): the
# small ones must keep all their bits too.  With a single nonzero product per sum the result is exact.
@pytest.mark.parametrize("split_k", [1, 3])
@pytest.mark.parametrize("lowest", [-149, -120])
def test_sgemm_small_values_beside_large_ones(P, split_k, lowest):
    K = 150
    eye = np.eye(K, dtype=np.float32)
    B = all_magnitudes(3, (K, 140), lowest)
    for v in split_tiles(P):
        v.split_k = split_k
        P.set_tile_override(v)
        for A, X, want in ((eye, B, B), (np.ascontiguousarray(B.T), eye, B.T)):
            C = dev(np.zeros(want.shape, np.float32))
            P.sgemm(dev(A), dev(X), C)
            assert np.array_equal(host(C), want), v
    P.set_tile_override(None)


def test_sgemm_large_value_meets_zero(P):
    # row 0 of A: 1 and tiny values in one thread's share; B has 0 where A has 1, large values elsewhere
    M, N, K = 70, 66, 130
    A, B, _ = synth.sgemm_inputs(M, N, K, seed=21)
    A[0] *= np.float32(2.0 ** -125)
    B *= np.float32(2.0 ** 120)
    A[0, ::8], B[::8] = 1.0, 0.0
    want = A.astype(np.float64) @ B.astype(np.float64)
    terms = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64)
    for v in split_tiles(P):
        P.set_tile_override(v)
        for a, b, w, t in ((A, B, want, terms), (B.T, A.T, want.T, terms.T)):
            C = dev(np.zeros(w.shape, np.float32))
            P.sgemm(dev(a), dev(b), C)
            assert (np.abs(host(C) - w) <= (K + 2) * 2.0 ** -24 * t).all(), v
    P.set_tile_override(None)


@pytest.mark.parametrize("s", CONV, ids=lambda s: s.name)
def test_conv_small_values_beside_large_ones(P, s):
    x = all_magnitudes(5, (s.N, s.C, s.H, s.W))
    pick = np.zeros((s.K, s.C, s.R, s.S), np.float32)
    for k in range(s.K):
        pick[k, k % s.C, s.R // 2, s.S // 2] = 1              # every output is one input value
    w = all_magnitudes(6, (s.K, s.C, s.R, s.S))
    dot = np.zeros((s.C, s.C, s.H, s.W), np.float32)
    for c in range(s.C):
        dot[c, c, s.H // 2, s.W // 2] = 1                     # every output is one filter value or zero
    for inp, f in ((x, pick), (dot, w)):
        want = conv64(inp, f, s.stride, s.pad)[0].astype(np.float32)
        dx, dw = dev(inp), dev(f)
        tap = P.filter_tap_copy(dw)
        for v in P.variants(0):
            if v.algo != 0 or v.bk != 16 or v.wm * v.wn > 64 * 64:
                continue
            for split_k, raster in ((1, 0), (2, 1), (1, 3)):
                for layout in ((0, 2) if s.C % 16 == 0 and 2 <= s.R * s.S <= 63 else (0,)):
                    v.split_k, v.raster, v.layout = split_k, raster, layout
                    P.set_tile_override(v)
                    got = host(P.conv2d_fwd(dx, dw, stride=s.stride, pad=s.pad, w_tap=tap if layout else None))
                    assert np.array_equal(got, want), v
    P.set_tile_override(None)


@pytest.mark.parametrize("s", [synth.ConvShape("c64", 2, 64, 9, 10, 128, 1, 1, 1, 0), synth.ConvShape("c32", 1, 32, 7, 6, 192, 1, 1, 1, 0),
                               synth.ConvShape("c16", 3, 16, 5, 4, 256, 1, 1, 1, 0)], ids=lambda s: s.name)
def test_pointwise_small_values_beside_large_ones(P, s):
    x = all_magnitudes(7, (s.N, s.C, s.H, s.W))
    pick = np.zeros((s.K, s.C, 1, 1), np.float32)
    pick[np.arange(s.K), np.arange(s.K) % s.C] = 1
    w = all_magnitudes(8, (s.K, s.C, 1, 1))
    dot = np.zeros((s.C, s.C, s.H, s.W), np.float32)
    dot[np.arange(s.C), np.arange(s.C), s.H // 2] = 1
    P.set_tile_override([v for v in P.variants(0) if v.algo == 2][0])
    for inp, f in ((x, pick), (dot, w)):
        got = host(P.conv2d_fwd(dev(inp), dev(f), stride=1, pad=0))
        assert np.array_equal(got, conv64(inp, f, 1, 0)[0].astype(np.float32))
    P.set_tile_override(None)


# The last channel of a reduction that does not fill its last stage: what lies past the end must not meet it.
@pytest.mark.parametrize("value", [np.inf, -np.inf])
@pytest.mark.parametrize("s", [s for s in CONV if s.R == 1] + [synth.ConvShape("c37", 2, 37, 6, 7, 40, 1, 1, 1, 0)], ids=lambda s: s.name)
def test_infinity_in_the_last_channel_stays_an_infinity(P, s, value):
    x, w, _ = synth.conv_inputs(s, seed=17, dist="normal")
    x[0, s.C - 1, 2, 2] = value
    want = conv64(x, w, s.stride, s.pad)[0]
    for v in P.variants(0):
        if v.algo != 0:
            continue
        for split_k in (1, 2):
            v.split_k = split_k
            P.set_tile_override(v)
            got = host(P.conv2d_fwd(dev(x), dev(w), stride=s.stride, pad=s.pad))
            inf = np.isinf(want)
            assert inf.any() and np.array_equal(got[inf], want[inf]) and np.isfinite(got[~inf]).all(), v
    P.set_tile_override(None)


@pytest.mark.parametrize("parts", [2, 3, 4, 5, 7, 8, 9, 13])
def test_sum_of_any_number_of_parts(P, parts):
    # the last part of a tile requests several parts together: counts at and beside its multiples; C is read, ragged rows.
    # Every part's length differs from the others' sum, so a part left out or counted twice shows.
    import torch
    g = np.random.default_rng(parts)
    M, N, K = 300, 141, 16 * 13 * 3 + 5
    A, B, C0 = (g.uniform(-1, 1, s).astype(np.float32) for s in ((M, K), (K, N), (M, N)))
    want = A.astype(np.float64) @ B + C0
    ab = np.abs(A).astype(np.float64) @ np.abs(B) + np.abs(C0)
    for v in P.variants(1):
        v.split_k, v.raster = parts, 1
        P.set_tile_override(v)
        first = host(P.sgemm(dev(A), dev(B), dev(C0)))
        # K fp32 roundings bound either instruction, two more for the parts' sum and C
        assert (np.abs(first - want) <= (K + parts + 2) * 2.0 ** -24 * ab).all(), v
        assert np.array_equal(first, host(P.sgemm(dev(A), dev(B), dev(C0)))), v
    P.set_tile_override(None)


# filters of 1, 3, 4, 9, 25, 31, 32, 49 and 63 taps: the row table repeats every so many stages; channel counts that end the
# reduction inside a stage and inside a period, parts that begin inside one and are shorter or longer than one
@pytest.mark.parametrize("R,S,C", [(1, 1, 160), (1, 3, 90), (2, 2, 61), (3, 3, 16), (3, 3, 83), (5, 5, 37), (1, 31, 6), (4, 8, 9), (7, 7, 21), (7, 9, 5)])
def test_row_table_of_any_reduction(P, R, S, C):
    s = synth.ConvShape("t", 2, C, 13, 17, 70, R, S, 1, min(R, S) // 2 + (R == S == 1))
    s = s if S <= 17 else synth.ConvShape("t", 2, C, 3, 40, 70, R, S, 2, 1)
    x, w, _ = synth.conv_inputs(s, seed=R * S + C, dist="normal")
    x[1, C - 1, 2, 3] = np.inf                    # the last channel's value reaches its own outputs only
    x[0, 0, 0, 0] = np.nan
    want, ab = conv64(x, w, s.stride, s.pad)
    dx, dw = dev(x), dev(w)
    fin = np.isfinite(want)
    for v in P.variants(0):
        if v.algo != 0 or v.bk != 16 or v.wm * v.wn > 64 * 64:
            continue
        for split_k in (1, 2, 5, 16):
            v.split_k, v.raster = split_k, 1
            P.set_tile_override(v)
            got = host(P.conv2d_fwd(dx, dw, stride=s.stride, pad=s.pad))
            assert np.array_equal(np.isnan(got), np.isnan(want)), v
            assert np.array_equal(got[~fin], want[~fin].astype(np.float32), equal_nan=True), v
            assert (np.abs(got[fin] - want[fin]) <= (C * R * S + 2) * 2.0 ** -24 * ab[fin]).all(), v
    P.set_tile_override(None)
