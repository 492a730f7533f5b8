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
    # The six products kept leave out less than 2^-25 of a product; every main accumulator step rounds once
    # per eight terms (<= 2^-24 of the running sum).  Worst case over the terms' magnitudes:
    # 2^-25 + (K/8 + 2) * 2^-24, plus the final rounding; fp32 in sequence would be allowed K * 2^-24.
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
