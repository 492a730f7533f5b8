// GEMM main loop with fp32 operands multiplied on the bfloat16 matrix cores.
//
// An fp32 value is the exact sum of three bfloat16 values (8 + 8 + 8 significand bits, each rounded
// to nearest): x = x0 + x1 + x2 (G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial
// Intelligence Datatype For Higher-Precision Computations", ARITH 2019).  Of the nine products of two such
// sums the six with weights down to 2^-18 are formed; the three left out together come to 2^-24 of the product
// at worst (1 + 2^-8 - 2^-17 squared), what one fp32 addition may round, and on uniform values to less than
// 2^-26 of it in 97 of 100.  v_mfma_f32_32x32x16_bf16 does 16 times the work per cycle of
// v_mfma_f32_32x32x2_f32, so six of them still leave 2.7 times the fp32 rate.
//
// Sums.  The products x0*y0 go to one accumulator, the five small ones to a second; both are added
// once at the end.  The main accumulator is then rounded twice per 16 reduction steps (the unit adds
// blocks of eight exact products at a time) where the fp32 instruction rounds 16 times.  Measured
// against 64 bits, relative 2-norm, normal inputs: reduction 64: 1.5e-7 -> 0.5e-7, 576: 4.4e-7 -> 1.3e-7,
// 4608: 11.8e-7 -> 4.2e-7; non-negative inputs the same factor.  (One accumulator for all six: no
// better than fp32; flushing it to a separate sum costs as many registers as the second one.)
//
// What the split cannot represent is recomputed with v_mfma_f32_32x32x2_f32 by the workgroup that meets
// it: infinities, NaN and values that round to a bfloat16 infinity leave a non-finite accumulator; a value
// below 2^-110 may have bits under 2^-133, the smallest bfloat16, which its third part drops.  The matrix
// unit itself keeps bfloat16 subnormals, so every value whose third part is exact is multiplied exactly.
#pragma once
#include "gemm_core.hpp"
#include <type_traits>

namespace polydl {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

#if defined(__HIP_DEVICE_COMPILE__)
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16(float x, float y)   // v_cvt_pk_bf16_f32, round to nearest even
{
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){x, y}, bf16x2));
}
__device__ __forceinline__ v16f mfma_bf16(u32x4 a, u32x4 b, v16f c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
#else   // the host pass has no bfloat16 vectors and only needs the signatures
__device__ inline uint32_t pack_bf16(float, float) { return 0; }
__device__ inline v16f mfma_bf16(u32x4, u32x4, v16f c) { return c; }
#endif

// LDS image of one stage of BK = 16 reduction rows: per operand and plane two runs (reduction 0-7 and
// 8-15) of 16-byte units, one unit per tile row / column, so a fragment is one 128-bit read whose 32
// lanes read 512 consecutive bytes.  Runs are PAD units apart so that the writers, which hold four or
// eight consecutive reduction values of a row, do not meet in the same banks.  Columns are permuted
// inside a wave's WN: column c lies at (c % NB)*(32 + SKEW) + c / NB, because block bj of a lane is the
// column NB*lane + bj (the epilogue stores NB adjacent columns as one vector).
template <class T>
struct SplitTile {
    static constexpr int SKEW = T::NB == 1 ? 0 : (T::NB == 2 ? 4 : 2);
    static constexpr int WCOLS = T::NB * (32 + SKEW);            // units a wave's WN columns take
    static constexpr int A_RUN = T::BM + 4, B_RUN = T::BN / T::WN * WCOLS + (T::NB == 1 ? 4 : 0);
    static constexpr int A_PLANE = 2 * A_RUN, B_PLANE = 2 * B_RUN;
    static constexpr int A_UNITS = 3 * A_PLANE, B_UNITS = 3 * B_PLANE;
    static constexpr int STAGE_UNITS = A_UNITS + B_UNITS;
    static constexpr int SPLIT_BYTES = 2 * STAGE_UNITS * 16;
    static constexpr int LDS_BYTES = SPLIT_BYTES > T::LDS_FLOATS * 4 ? SPLIT_BYTES : T::LDS_FLOATS * 4;
    static __device__ __forceinline__ int col_pos(int c)
    {
        const int w = c / T::WN, r = c % T::WN;
        return w * WCOLS + (r % T::NB) * (32 + SKEW) + r / T::NB;
    }
};

// true if bits (OR of the bit patterns of the second remainders, see SplitUnit) shows a value whose three
// parts do not add up to it.  What is left of a value after two parts has at most seven significant bits and is
// the third part, unless some of them lie below 2^-133; a float32 is a bfloat16 exactly where its low
// sixteen bits are zero, for subnormal numbers too.
__device__ __forceinline__ bool split_lossy(uint32_t bits) { return (bits & 0xFFFFu) != 0; }

// RPT (4 or 8) consecutive reduction values of one row on their way into the three planes.  The splitting
// goes in steps of about five vector instructions, three per pair of values, so that the main loop can
// deal them out between its matrix instructions.
template <int RPT>
struct SplitUnit {
    static constexpr int STEPS = 3 * RPT / 2;
    uint32_t p[3][RPT / 2];
    float rx, ry;
    uint32_t seen = 0;        // OR of the bit patterns of what every value left for its third part
    template <int STEP>
    __device__ __forceinline__ void step(const float *v)
    {
        constexpr int i = STEP / 3, PHASE = STEP % 3;
        if constexpr (PHASE == 0) {
            p[0][i] = pack_bf16(v[2 * i], v[2 * i + 1]);
            rx = v[2 * i] - __builtin_bit_cast(float, p[0][i] << 16);
            ry = v[2 * i + 1] - __builtin_bit_cast(float, p[0][i] & 0xFFFF0000u);
        } else if constexpr (PHASE == 1) {
            p[1][i] = pack_bf16(rx, ry);
            rx -= __builtin_bit_cast(float, p[1][i] << 16);
            ry -= __builtin_bit_cast(float, p[1][i] & 0xFFFF0000u);
        } else {
            p[2][i] = pack_bf16(rx, ry);
            // as an instruction of its own place: the compiler would gather the ORs of a whole stage at
            // the first use and wait there for loads that are needed much later
            asm volatile("v_or3_b32 %0, %1, %2, %0" : "+v"(seen) : "v"(rx), "v"(ry));
        }
    }
    // base: first unit of the operand's stage; k_in: reduction index of the first value inside the stage
    __device__ __forceinline__ void write(u32x4 *base, int plane, int run, int pos, int k_in) const
    {
        u32x4 *u = base + (k_in >> 3) * run + pos;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            if constexpr (RPT == 8) u[i * plane] = (u32x4){p[i][0], p[i][1], p[i][2], p[i][3]};
            else *(reinterpret_cast<u32x2 *>(u + i * plane) + ((k_in >> 2) & 1)) = (u32x2){p[i][0], p[i][1]};
        }
    }
};

// calls f with the compile-time integers FROM .. TO-1
template <int FROM, int TO, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    if constexpr (FROM < TO) {
        f(std::integral_constant<int, FROM>{});
        static_for<FROM + 1, TO>(f);
    }
}

// Fragments of a stage and their products.
template <class T>
struct SplitAcc {
    v16f hi[T::MB][T::NB], lo[T::MB][T::NB];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
                for (int r = 0; r < 16; ++r) { hi[bi][bj][r] = 0.f; lo[bi][bj][r] = 0.f; }
    }
    // acc = hi + lo; true if any sum of this lane is not finite
    __device__ __forceinline__ bool finish(v16f (&acc)[T::MB][T::NB]) const
    {
        float f = 0.f;
#pragma unroll
        for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    acc[bi][bj][r] = hi[bi][bj][r] + lo[bi][bj][r];
                    f = __builtin_fmaf(acc[bi][bj][r], 0.f, f);
                }
        return !(f == 0.f);
    }
};

// The operands of a stage a wave multiplies: planes 0..2 of its row and column blocks.
template <class T>
struct SplitFrags {
    typedef SplitTile<T> L;
    u32x4 a[3][T::MB], b[3][T::NB];
    // stage: first unit of the stage's LDS image
    template <int PLANE>
    __device__ __forceinline__ void read_a(const u32x4 *stage, int wm0, int lane)
    {
#pragma unroll
        for (int bi = 0; bi < T::MB; ++bi)
            a[PLANE][bi] = stage[PLANE * L::A_PLANE + (lane >> 5) * L::A_RUN + wm0 + 32 * bi + (lane & 31)];
    }
    template <int PLANE>
    __device__ __forceinline__ void read_b(const u32x4 *stage, int wave_col, int lane)
    {
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj)
            b[PLANE][bj] = stage[L::A_UNITS + PLANE * L::B_PLANE + (lane >> 5) * L::B_RUN + wave_col * L::WCOLS +
                                 bj * (32 + L::SKEW) + (lane & 31)];
    }
    template <int PA, int PB>
    __device__ __forceinline__ void mma(v16f (&acc)[T::MB][T::NB], int block) const
    {
        const int bi = block / T::NB, bj = block % T::NB;
        acc[bi][bj] = mfma_bf16(a[PA][bi], b[PB][bj], acc[bi][bj]);
    }
};

// ---- A operand: row-major [Mg][lda], reduction index contiguous ------------------------------
// A thread owns RPT consecutive reduction values of one row of every stage (a whole unit where the tile has
// enough rows for all threads), fetched with 128-bit loads.  Buffer loads only need dword alignment, so rows
// of any length and base do; values past the end of the reduction (last stage only) are zeroed.
template <class T>
struct SplitALoader {
    typedef SplitTile<T> L;
    static constexpr int RPT = T::BM * T::BK / T::NT, TPR = T::BK / RPT, VECS = RPT / 4;
    static_assert((RPT == 4 || RPT == 8) && T::BK == 16, "a quad or an octet per thread");
    const float *base;
    uint64_t bytes;
    float regs[2][RPT];
    SplitUnit<RPT> unit;
    uint32_t off0;
    int row, k_in;

    __device__ __forceinline__ void init(const float *A, int tid, int m0, int Mg, int Kg, int lda)
    {
        base = A + (size_t)m0 * lda;
        bytes = ((size_t)(Mg - m0 - 1) * lda + Kg) * 4;
        row = tid / TPR;
        k_in = tid % TPR * RPT;
        off0 = m0 + row < Mg ? ((uint32_t)row * (uint32_t)lda + (uint32_t)k_in) * 4u : kOobOffset;
    }
    template <int SET, bool FULL>
    __device__ __forceinline__ void load(int k0, int kend)
    {
        const int kb = FULL || k0 < kend ? k0 : 0;   // past the end every lane reads out of range: keep the base inside A
        __amdgpu_buffer_rsrc_t rsrc = make_rsrc(base + kb, bytes - (uint64_t)kb * 4);
        const int krem = kend - k0;
#pragma unroll
        for (int i = 0; i < VECS; ++i) {
            v4f v = buf_load4(rsrc, FULL || k_in + 4 * i < krem ? off0 + 16u * i : kOobOffset);
#pragma unroll
            for (int j = 0; j < 4; ++j) regs[SET][4 * i + j] = FULL || k_in + 4 * i + j < krem ? v[j] : 0.f;
        }
    }
    template <int SET, int STEP>
    __device__ __forceinline__ void step() { unit.template step<STEP>(regs[SET]); }
    __device__ __forceinline__ void write(u32x4 *stage) const { unit.write(stage, L::A_PLANE, L::A_RUN, row, k_in); }
    __device__ __forceinline__ bool lossy() const { return split_lossy(unit.seen); }
};

// ---- B operand of a plain GEMM: row-major [Kg][ldb], column index contiguous ------------------
// A thread owns one column of the tile and RPT consecutive reduction rows of every stage; a wave's lanes
// read 256 consecutive bytes per row.
template <class T>
struct SplitBLoaderRows {
    typedef SplitTile<T> L;
    static constexpr int GROUPS = T::NT / T::BN, RPT = T::BK / GROUPS;
    static_assert(T::NT % T::BN == 0 && T::BN % 64 == 0 && (RPT == 4 || RPT == 8), "one column per thread");
    const float *base;
    int Kg, ldb, ncols;
    float regs[2][RPT];
    SplitUnit<RPT> unit;
    uint32_t off0;
    int pos, row0;
    __amdgpu_buffer_rsrc_t rsrc;   // of the stage being fetched
    int krem;

    __device__ __forceinline__ void init(const float *B, int tid, int n0, int Ng, int Kg_, int ldb_)
    {
        base = B + n0;
        Kg = Kg_;
        ldb = ldb_;
        ncols = Ng - n0;
        const int col = tid % T::BN;
        row0 = __builtin_amdgcn_readfirstlane(tid / T::BN) * RPT;
        off0 = n0 + col < Ng ? 4u * (uint32_t)col : kOobOffset;
        pos = L::col_pos(col);
    }
    // a stage is fetched row by row: begin() once, then row<0 .. RPT-1>()
    template <bool FULL>
    __device__ __forceinline__ void begin(int k0, int kend)
    {
        const int kb = FULL || k0 < kend ? k0 : 0;
        rsrc = make_rsrc(base + (size_t)kb * ldb, ((uint64_t)(Kg - kb - 1) * ldb + ncols) * 4);
        krem = kend - k0;
    }
    template <int SET, bool FULL, int J>
    __device__ __forceinline__ void row()
    {
        // the range check does not see the uniform offset: rows past the end are switched off per lane
        const bool ok = FULL || row0 + J < krem;
        regs[SET][J] = buf_load1(rsrc, ok ? off0 : kOobOffset, (uint32_t)(ok ? row0 + J : 0) * ((uint32_t)ldb * 4u));
    }
    template <int SET, int STEP>
    __device__ __forceinline__ void step() { unit.template step<STEP>(regs[SET]); }
    __device__ __forceinline__ void write(u32x4 *stage) const
    {
        unit.write(stage + L::A_UNITS, L::B_PLANE, L::B_RUN, pos, row0);
    }
    __device__ __forceinline__ bool lossy() const { return split_lossy(unit.seen); }
};

// Software pipeline.  While stage t is multiplied out of LDS buffer t&1, stage t+1 is split from registers into
// the other buffer: A first, whose registers then take the loads of stage t+3, then B, whose other register
// set takes stage t+2 at the stage's start -- every load has one and a half stages to come back.  One
// barrier per stage.  About six vector instructions are free behind each matrix instruction if they are
// dealt out between them; left alone, the compiler gathers the splitting behind the last one and the loads
// at the end, so every step is fenced (2048^3, 128x128 tile: 115 -> 99 us).  A longer pipeline that keeps half
// of a stage's products for after the barrier, so that no fragment read is waited for, measured the same on
// large products and 2-5 % slower on small ones (its prologue is a stage longer).
// FULL: the stages the loads fetch lie wholly inside the reduction (no test per load).
template <class T, int HALF, bool FULL, class AL, class BL>
__device__ __forceinline__ void split_stage(u32x4 *lds, AL &al, BL &bl, SplitAcc<T> &acc, int k, int kend, int tid,
                                            int wm0, int wave_col)
{
    typedef SplitTile<T> L;
    constexpr int BK = T::BK, BLOCKS = T::MB * T::NB, MM = 6 * BLOCKS;
    constexpr int SA = 3 * AL::RPT / 2, SB = 3 * BL::RPT / 2, SPREAD = MM - MM / 6;   // the writes end before the barrier
    const int lane = tid & 63;
    const u32x4 *cur = lds + HALF * L::STAGE_UNITS;
    u32x4 *next = lds + (HALF ^ 1) * L::STAGE_UNITS;
    SplitFrags<T> f;
    f.template read_a<0>(cur, wm0, lane);
    f.template read_b<0>(cur, wave_col, lane);
    f.template read_a<1>(cur, wm0, lane);
    f.template read_b<1>(cur, wave_col, lane);
    f.template read_a<2>(cur, wm0, lane);
    f.template read_b<2>(cur, wave_col, lane);
    bl.template begin<FULL>(k + 2 * BK, kend);
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, MM>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, P = i / BLOCKS, blk = i % BLOCKS;
        if constexpr (P == 0) f.template mma<0, 0>(acc.hi, blk);
        if constexpr (P == 1) f.template mma<1, 0>(acc.lo, blk);
        if constexpr (P == 2) f.template mma<0, 1>(acc.lo, blk);
        if constexpr (P == 3) f.template mma<1, 1>(acc.lo, blk);
        if constexpr (P == 4) f.template mma<2, 0>(acc.lo, blk);
        if constexpr (P == 5) f.template mma<0, 2>(acc.lo, blk);
        // loads of stage t+2's B rows, spread over the first half
        static_for<i * BL::RPT * 2 / MM, (i + 1) * BL::RPT * 2 / MM>([&](auto j) __attribute__((always_inline)) {
            if constexpr (decltype(j)::value < BL::RPT) bl.template row<HALF, FULL, decltype(j)::value>();
        });
        constexpr int S0 = i * (SA + SB) / SPREAD, S1 = (i + 1) * (SA + SB) / SPREAD;
        static_for<S0 < SA + SB ? S0 : SA + SB, S1 < SA + SB ? S1 : SA + SB>([&](auto sc) __attribute__((always_inline)) {
            constexpr int st = decltype(sc)::value;
            if constexpr (st < SA) al.template step<HALF ^ 1, st>();
            else bl.template step<HALF ^ 1, st - SA>();
            if constexpr (st == SA - 1) {
                al.write(next);
                al.template load<HALF ^ 1, FULL>(k + 3 * BK, kend);
            }
            if constexpr (st == SA + SB - 1) bl.write(next);
        });
        __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
}

template <class T, class AL, class BL>
__device__ __forceinline__ void split_mainloop(u32x4 *lds, AL &al, BL &bl, SplitAcc<T> &acc, int kbegin, int kend,
                                               int tid, int wm0, int wave_col)
{
    constexpr int BK = T::BK, SA = 3 * AL::RPT / 2, SB = 3 * BL::RPT / 2;
    auto load_b = [&](auto set, int k0) __attribute__((always_inline)) {
        bl.template begin<false>(k0, kend);
        static_for<0, BL::RPT>([&](auto j) __attribute__((always_inline)) {
            bl.template row<decltype(set)::value, false, decltype(j)::value>();
        });
    };
    al.template load<0, false>(kbegin, kend);
    load_b(std::integral_constant<int, 0>{}, kbegin);
    al.template load<1, false>(kbegin + BK, kend);
    load_b(std::integral_constant<int, 1>{}, kbegin + BK);
    static_for<0, SA>([&](auto j) __attribute__((always_inline)) { al.template step<0, decltype(j)::value>(); });
    al.write(lds);
    al.template load<0, false>(kbegin + 2 * BK, kend);
    static_for<0, SB>([&](auto j) __attribute__((always_inline)) { bl.template step<0, decltype(j)::value>(); });
    bl.write(lds);
    __syncthreads();
    int k0 = kbegin;
    for (; k0 + 5 * BK <= kend; k0 += 2 * BK) {
        split_stage<T, 0, true>(lds, al, bl, acc, k0, kend, tid, wm0, wave_col);
        split_stage<T, 1, true>(lds, al, bl, acc, k0 + BK, kend, tid, wm0, wave_col);
    }
    // at most five stages are left
    for (; k0 + BK < kend; k0 += 2 * BK) {
        split_stage<T, 0, false>(lds, al, bl, acc, k0, kend, tid, wm0, wave_col);
        split_stage<T, 1, false>(lds, al, bl, acc, k0 + BK, kend, tid, wm0, wave_col);
    }
    if (k0 < kend) split_stage<T, 0, false>(lds, al, bl, acc, k0, kend, tid, wm0, wave_col);   // workgroup-uniform
}

}  // namespace polydl
