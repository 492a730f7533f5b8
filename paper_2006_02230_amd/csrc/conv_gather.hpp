// What the convolution kernels that view the layer as an implicit GEMM share: launch arguments, the im2col
// gather, the tile a workgroup takes, and what follows the reduction.
#pragma once
#include "gemm_core.hpp"
#include "internal.hpp"
#include "split_core.hpp"

namespace polydl {

struct ConvKArgs {
    const float *in, *wt, *bias;
    float *out;
    int C, H, W, K, R, S, stride, pad, P, Q;
    int PQ, RS, HW, CHW;
    int Kg, Ng;                 // reduction length C*R*S, number of output pixels N*P*Q
    uint32_t magic_C;           // GATHER_TAPMAJOR: exact division of a reduction index by C (C > 1)
    uint32_t magic_RS, magic_S; // exact division of a reduction index by R*S and by S,
    uint32_t one_RS, one_S;     // see fast_div(): magic multiplier and the all-ones mask for d == 1
    uint32_t recip_PQ, recip_Q; // for div_by(): pixel index -> (image, row, column)
    uint64_t in_bytes, out_bytes;
    int tiles_m, tiles_n;
    int split_k, k_per_split;
    // tail_parts > 1: one-dimensional grid; the first whole_tiles tiles run their reduction whole,
    // each later tile in tail_parts parts of tail_k reduction elements
    int whole_tiles, tail_parts, tail_k;
    uint32_t recip_tail;
    int raster, act;
    int pre_act;                // activation applied to every input element as its stage is filled
    float *partials;            // split_k > 1: [tile][part][BM*BN] accumulator tiles in register order
    unsigned *counters;         // split_k > 1: per tile, how many of its reduction parts have finished
};

// ---- B operand: on-the-fly im2col gather from NCHW --------------------------------------------
// A thread owns one output pixel (one column of the stage) for the whole reduction; per stage it
// loads BK / (NT/BN) reduction rows of that column.  The reduction row is the same for all lanes
// of a wave, so its split into (c, r, s) is scalar work.  Whether tap (r, s) falls inside the
// image for this pixel is kept as one bit per filter row and per filter column.
// n / d without a branch: (n * magic) >> 32 is exact for n*d < 2^32 when d > 1; for d == 1 the
// magic is 0 and the all-ones mask passes n through.
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t magic, uint32_t ones_if_d1)
{
    return __umulhi(n, magic) + (n & ones_if_d1);
}

// The n lowest bits, 0 <= n <= MAX (31 or 32).  In 32 bits: see "The order of a table's entry" below.  A bit field mask, and for n = 32,
// whose low five bits are 0, bit 5 spread over the word: one and three instructions, no compare (with compare and select
// the prologue of small layers was 0.05 .. 0.1 us longer: one 64 -> 64 3x3 image 11.01 -> 11.06 us).
template <int MAX = 32>
__device__ __forceinline__ uint32_t low_bits(int n)
{
    const uint32_t m = (1u << (n & 31)) - 1u;
    return MAX < 32 ? m : m | (uint32_t)((int)((uint32_t)n << 26) >> 31);
}
// Bits i of 0 .. n-1 with i < lo or i >= hi (n <= MAX).
template <int MAX = 32>
__device__ __forceinline__ uint32_t outside_bits(int lo, int hi, int n)
{
    lo = min(max(lo, 0), n);
    hi = min(max(hi, 0), n);
    return low_bits<MAX>(lo) | (low_bits<MAX>(n) & ~low_bits<MAX>(hi));
}

// How a load finds its element and whether it lies inside the image:
//  GATHER_ANY   any filter: per-lane row and column bit masks, offset built per lane;
//  GATHER_POINT 1x1 filters without padding: reduction row k is channel k and every tap lies inside
//               the image, so the lane keeps the byte offset of its pixel and the channel offset
//               rides in the instruction's uniform offset -- no per-lane arithmetic per load;
//  GATHER_TAPS1 / GATHER_TAPS2  filters of at most 31 / 63 taps: the lane keeps one bit per tap
//               (set: outside the image) in one / two registers and the byte offset of tap (0,0);
//               the tap's distance is uniform and rides in the uniform offset, so a load costs a
//               bit extract and a merge of that bit into the top of the offset.
//  GATHER_TAPMAJOR  filters of 2 .. 63 taps whose channel count is a multiple of the stage depth, with
//               a second copy of the filter in the blocked layout [K][R][S][C] (KCRSck with
//               bc = C, bk = 1): the reduction is walked tap by tap, all channels of a tap before
//               the next tap (the order is free, section "Microkernel Specification"), so a whole
//               stage shares one tap: its validity bit and its distance are found once per stage,
//               not per element, and the channel rides in the uniform offset.  In that copy the
//               filter rows are contiguous in the walked order, so they load as in a plain GEMM.
//  GATHER_TABLE  filters of at most 63 taps with a short reduction (gather_table_fits()), on the fp32
//               instruction: as GATHER_TAPS2, but the (c, r, s) split of a reduction row is not
//               redone by every wave for every element.  The workgroup writes (tap number, distance of the
//               row's tap and channel in bytes) of every row into LDS once; a load then
//               reads its row's entry (one address per stage, constant offsets), adds the distance
//               to the lane's offset and shifts the lane's 64 tap bits by the tap number.  Same
//               vector instructions per element as GATHER_TAPS2, a tenth of its scalar ones: the one
//               scalar unit of a compute unit serves four SIMDs, and at 18 scalar instructions per
//               matrix instruction (the stem layer) it, not the matrix cores, set the pace.
//  With SPLIT, GATHER_TAPS1 / GATHER_TAPS2 read their rows from a table as well, of any reduction's length: a stage is 16
//               rows, so the rows' taps repeat every R*S stages, 16 channels further on.  The table holds one such period
//               (or a part's stages, if fewer), the 16 channels per period ride in the uniform offset, and only the
//               stage number is divided, once per stage.  Batch 32 with the filter in KCRS order only: 512 -> 512 3x3
//               on 7x7 70.1 -> 64.4 us (8.4 scalar instructions per matrix instruction before), 83 -> 201 3x3 on 35x29,
//               batch 7, 30.8 -> 28.6, one 64 -> 64 3x3 image 12.1 -> 11.05.
//  The order of a table's entry: the tap number, by which the lane's 64 tap bits are shifted, comes first.  An entry is read into
//               an aligned pair of registers, so the amount of the shift lies in an even one.  In the odd one it can be the last
//               register of the kernel's allocation, and there gfx950 shifts by another wave's value now and then (measured
//               on a full card: a quarter of such shifts); the compiler knows that of gfx90a only.  With the distance
//               first, 3 -> 512 5x5 on 28x15 read taps outside the image as soon as the fp32 kernel took 72 registers.
//               tests/test_device_code.py looks for such shifts in the built library.
enum { GATHER_ANY = 0, GATHER_POINT = 1, GATHER_TAPS1 = 2, GATHER_TAPS2 = 3, GATHER_TAPMAJOR = 4, GATHER_TABLE = 5 };


// SPLIT: the stage goes to LDS as three bfloat16 planes (split_core.hpp), so a thread's rows of a stage are
// consecutive; otherwise they lie KSTEP apart.  KTAIL: the reduction may end inside a stage (GATHER_POINT only,
// every other mode tests each row anyway).
template <class T, int MODE, bool SPLIT = false, bool KTAIL = true>
struct BLoaderIm2col {
    typedef SplitTile<T> L;
    static constexpr bool POINT = MODE == GATHER_POINT;
    static constexpr bool TAPMAJOR = MODE == GATHER_TAPMAJOR;
    static constexpr bool TABLE = MODE == GATHER_TABLE;
    static constexpr bool TAPS = MODE == GATHER_TAPS1 || MODE == GATHER_TAPS2 || TAPMAJOR || TABLE;
    static constexpr int LAST_BIT = MODE == GATHER_TAPS1 ? 31 : 63;   // never a tap: always set
    static constexpr int KSTEP = T::NT / T::BN;  // reduction rows covered by one pass of the workgroup
    static constexpr int ITERS = T::BK / KSTEP;
    static_assert(T::BK % KSTEP == 0, "stage depth must be a multiple of the rows loaded per pass");
    static_assert(!SPLIT || ITERS == 4 || ITERS == 8, "whole quads");
    static constexpr int RPT = ITERS;
    static constexpr bool PERIODIC = SPLIT && (MODE == GATHER_TAPS1 || MODE == GATHER_TAPS2);
    static constexpr int TABLE_ROWS = PERIODIC ? (LAST_BIT + 2) * 16 : MODE == GATHER_TABLE ? kTableRows : 1;
    static_assert(!PERIODIC || T::BK == 16, "a period is R*S stages of 16 rows");
    SplitUnit<SPLIT ? RPT : 4> unit;                                 // SPLIT: the values on their way into the planes
    float regs[2][ITERS];
    __amdgpu_buffer_rsrc_t rsrc;
    int pix_off;      // element offset of tap (0,0), channel 0 of this pixel from the descriptor base
    uint32_t rmask, smask;   // GATHER_TAPS*: the tap bits 0-31 and 32-63
    int krow0, lds_off;
    int RS, S, HW, W, pre_act, C;
    uint32_t magic_RS, magic_S, one_RS, one_S, magic_C;
    const uint2 *tab;   // GATHER_TABLE, PERIODIC: per reduction row (tap number, byte distance), in LDS

    // GATHER_TABLE: the workgroup fills the table (rows at or past the end of the reduction get the
    // bit that is always set); the caller puts a barrier between this and the first load.
    // PERIODIC: the rows of the part's stages, at most one period; behind that the last stage as it ends, and one of
    // rows that lie outside, for the loads that run ahead.
    __device__ __forceinline__ void fill_table(const ConvKArgs &p, int tid, uint2 *t, int kbegin, int kend)
    {
        tab = t;
        if constexpr (PERIODIC) {
            const uint32_t period = (uint32_t)p.RS * 16u;
            auto phase_row = [&](int k) __attribute__((always_inline)) {   // of the stage that begins at row k (uniform)
                const uint32_t st = (uint32_t)k >> 4;
                return (st - fast_div(st, p.magic_RS, p.one_RS) * (uint32_t)p.RS) * 16u;
            };
            const int last = (kend - 1) & ~15;
            const uint32_t first = phase_row(kbegin), first_of_last = phase_row(last);
            const uint32_t rows = min((uint32_t)(last - kbegin) + 16u, period);
            for (uint32_t e = tid; e < rows + 32u; e += T::NT) {
                uint32_t row = first + e, at;
                if (row >= period) row -= period;
                at = row;
                bool in = true;
                if (e >= rows) {      // behind the period: the last stage once more, its rows past kend outside, and a stage of such rows
                    row = first_of_last + ((e - rows) & 15u);
                    at = period + (e - rows);
                    in = last + (int)(e - rows) < kend;
                }
                const uint32_t c = fast_div(row, p.magic_RS, p.one_RS), rs = row - c * (uint32_t)p.RS;
                const uint32_t r = fast_div(rs, p.magic_S, p.one_S), sx = rs - r * (uint32_t)p.S;
                t[at] = (uint2){in ? rs : (uint32_t)LAST_BIT, (c * (uint32_t)p.HW + r * (uint32_t)p.W + sx) * 4u};
            }
        }
        if constexpr (TABLE) {
            // every row a load can ask for: the reduction rounded up to whole stages and the two
            // stages the loads run ahead (the launcher checked that the table holds them)
            const int rows = ((p.Kg + T::BK - 1) / T::BK + 2) * T::BK;
            for (int kg = tid; kg < rows; kg += T::NT) {
                uint2 e = {(uint32_t)LAST_BIT, 0u};
                if (kg < p.Kg) {
                    const uint32_t c = fast_div((uint32_t)kg, p.magic_RS, p.one_RS), rs = (uint32_t)kg - c * (uint32_t)p.RS;
                    const uint32_t r = fast_div(rs, p.magic_S, p.one_S), sx = rs - r * (uint32_t)p.S;
                    e.x = rs;
                    e.y = (c * (uint32_t)p.HW + r * (uint32_t)p.W + sx) * 4u;
                }
                t[kg] = e;
            }
        }
    }

    __device__ __forceinline__ void init(const ConvKArgs &p, int tid, int n0)
    {
        RS = p.RS; S = p.S; HW = p.HW; W = p.W; pre_act = p.pre_act; C = p.C; magic_C = p.magic_C;
        magic_RS = p.magic_RS; magic_S = p.magic_S; one_RS = p.one_RS; one_S = p.one_S;
        const int col = tid % T::BN;
        krow0 = __builtin_amdgcn_readfirstlane(tid / T::BN) * (SPLIT ? ITERS : 1);
        lds_off = SPLIT ? L::col_pos(col) : krow0 * T::LDB + col;
        // the descriptor starts at the first image this tile touches: offsets stay small
        uint32_t rem0;
        const int img0 = (int)div_by((uint32_t)n0, (uint32_t)p.PQ, p.recip_PQ, rem0);
        const uint64_t skip = (uint64_t)img0 * p.CHW * 4;
        // GATHER_TAPS*: per-lane offsets are those of tap (0,0), which lies up to pad rows and pad
        // columns before the image; the descriptor starts that much earlier so that they are not
        // negative (no load is made there: such taps are flagged outside)
        const int lead = TAPS ? (p.pad * p.W + p.pad) * 4 : 0;
        rsrc = make_rsrc(reinterpret_cast<const char *>(p.in) + skip - lead, p.in_bytes - skip + lead);
        const int colg = n0 + col;
        rmask = 0; smask = 0; pix_off = 0;
        if (colg < p.Ng) {
            uint32_t pq, oq;
            int img = (int)div_by((uint32_t)colg, (uint32_t)p.PQ, p.recip_PQ, pq);
            int op = (int)div_by(pq, (uint32_t)p.Q, p.recip_Q, oq);
            int ih0 = op * p.stride - p.pad, iw0 = (int)oq * p.stride - p.pad;
            pix_off = (img - img0) * p.CHW + ih0 * p.W + iw0;
            // filter rows r < -ih0 or r >= H - ih0 and columns s < -iw0 or s >= W - iw0 fall outside
            constexpr int MAX = MODE == GATHER_TAPS1 ? 31 : 32;
            const uint32_t rows_out = outside_bits<MAX>(-ih0, p.H - ih0, p.R);
            const uint32_t cols_out = outside_bits<MAX>(-iw0, p.W - iw0, p.S);
            if constexpr (MODE == GATHER_ANY) {
                rmask = ~rows_out;
                smask = ~cols_out;
            }
            if constexpr (TAPS) {
                const uint32_t all_cols = low_bits<MAX>(p.S);
                uint64_t taps = 0;
                for (int r = 0; r < p.R; ++r)
                    taps |= (uint64_t)((rows_out >> r) & 1u ? all_cols : cols_out) << (r * p.S);
                rmask = (uint32_t)taps;
                smask = (uint32_t)(taps >> 32);
                pix_off = pix_off * 4 + lead;
            }
        } else if constexpr (TAPS) {
            rmask = 0xFFFFFFFFu; smask = 0xFFFFFFFFu;
        }
        if constexpr (TAPS) { if (MODE == GATHER_TAPS1) rmask |= 1u << 31; else smask |= 1u << 31; }
        (void)C; (void)magic_C;
        if constexpr (POINT) pix_off = colg < p.Ng ? pix_off * 4 : (int)kOobOffset;   // bytes, or out of range
    }
    // element of reduction row kg (wave-uniform), its split into (c, r, s) done here
    template <bool FULL>
    __device__ __forceinline__ float gather(uint32_t kg, int kend) const
    {
        uint32_t c = fast_div(kg, magic_RS, one_RS);
        uint32_t rs = kg - c * (uint32_t)RS;
        uint32_t r = fast_div(rs, magic_S, one_S);
        uint32_t s = rs - r * (uint32_t)S;
        int koff = (int)c * HW + (int)r * W + (int)s;
        if constexpr (TAPS) {
            // a row at or past kend takes the bit that is always set
            const uint32_t t = FULL || (int)kg < kend ? rs : (uint32_t)LAST_BIT;
            uint32_t word = rmask;
            if constexpr (MODE == GATHER_TAPS2) word = t < 32u ? rmask : smask;
            const uint32_t outside = (word >> (t & 31u)) & 1u;
            return buf_load1(rsrc, (uint32_t)pix_off | (outside << 31), (uint32_t)koff * 4u);
        }
        uint32_t ok = (uint32_t)(FULL || (int)kg < kend) & (rmask >> r) & (smask >> s) & 1u;
        // not ok -> set the top bit: at or beyond 2^31 every descriptor reads as zero
        return buf_load1(rsrc, ((uint32_t)(pix_off + koff) * 4u) | ((ok ^ 1u) << 31));
    }
    template <int SET>
    __device__ __forceinline__ void load(int k0, int kend)
    {
        if constexpr (POINT) {
            // A row at or past kend (wave-uniform) meets zeros in the filter operand.  In a stage that is
            // multiplied it must read as zero, not as a value of another channel, which may be an infinity;
            // where the reduction is whole stages it only has to stay inside the tensor.
#pragma unroll
            for (int i = 0; i < ITERS; ++i) {
                const int kg = k0 + krow0 + i * KSTEP;
                if constexpr (KTAIL)
                    regs[SET][i] = buf_load1(rsrc, (uint32_t)pix_off | (kg < kend ? 0u : kOobOffset), (uint32_t)(kg * HW) * 4u);
                else regs[SET][i] = buf_load1(rsrc, (uint32_t)pix_off, (uint32_t)(min(kg, kend - 1) * HW) * 4u);
            }
            return;
        }
        if constexpr (TAPMAJOR) {
            // one tap for the whole stage: its bit and its distance once, the channel in the uniform offset
            const uint32_t kk = k0 < kend ? (uint32_t)k0 : 0u;
            const uint32_t tap = __umulhi(kk, magic_C), c0 = kk - tap * (uint32_t)C;
            const uint32_t r = fast_div(tap, magic_S, one_S), sx = tap - r * (uint32_t)S;
            const uint32_t t = k0 < kend ? tap : (uint32_t)LAST_BIT;
            const uint32_t word = t < 32u ? rmask : smask;
            const uint32_t off = (uint32_t)pix_off | (((word >> (t & 31u)) & 1u) << 31);
            uint32_t koff = ((c0 + (uint32_t)krow0) * (uint32_t)HW + r * (uint32_t)W + sx) * 4u;
#pragma unroll
            for (int i = 0; i < ITERS; ++i) {
                regs[SET][i] = buf_load1(rsrc, off, koff);
                koff += (uint32_t)(KSTEP * HW) * 4u;
            }
            return;
        }
        if constexpr (TABLE) {
            // one LDS address per stage; the rows of this thread lie KSTEP entries apart.  Rows at or
            // past kend are either past the reduction's end (entry: always outside) or belong to a
            // look-ahead stage of a split reduction, whose values are never multiplied.
            const uint2 *row = tab + (k0 + krow0);
            const uint64_t taps = ((uint64_t)smask << 32) | rmask;
#pragma unroll
            for (int i = 0; i < ITERS; ++i) {
                const uint2 e = row[i * KSTEP];
                const uint32_t outside = (uint32_t)(taps >> e.x);      // bit 0 counts: the shift below drops the rest
                regs[SET][i] = buf_load1(rsrc, ((uint32_t)pix_off + e.y) | (outside << 31));
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < ITERS; ++i) regs[SET][i] = gather<false>((uint32_t)(k0 + krow0 + i * KSTEP), kend);
    }
    // The element-wise operator that precedes the convolution is applied where its operand is
    // first touched (the symmetric case of section "Operator Fusion": fused with the first iteration
    // of the heavy operator's reduction loops); zero fill stays zero under ReLU and ReLU6.
    template <int SET>
    __device__ __forceinline__ void activate()
    {
        if (pre_act != POLYDL_ACT_NONE) {   // uniform
#pragma unroll
            for (int i = 0; i < ITERS; ++i) {
                float v = fmaxf(regs[SET][i], 0.f);
                regs[SET][i] = pre_act == POLYDL_ACT_RELU6 ? fminf(v, 6.f) : v;
            }
        }
    }
    // the steps of split_core.hpp's main loop; a stage is fetched row by row
    int s_k0, s_kend;
    uint32_t s_off, s_koff;          // GATHER_TAPMAJOR: the stage's lane offset and first row's distance; PERIODIC: its period's distance
    const uint2 *s_row;              // PERIODIC: the stage's first entry
    template <bool FULL>
    __device__ __forceinline__ void begin(int k0, int kend)
    {
        s_k0 = k0; s_kend = kend;
        if constexpr (TAPMAJOR) {
            // one tap for the whole stage: its bit and its distance once, the channel in the uniform offset
            const uint32_t kk = FULL || k0 < kend ? (uint32_t)k0 : 0u;
            const uint32_t tap = __umulhi(kk, magic_C), c0 = kk - tap * (uint32_t)C;
            const uint32_t r = fast_div(tap, magic_S, one_S), sx = tap - r * (uint32_t)S;
            const uint32_t t = FULL || k0 < kend ? tap : (uint32_t)LAST_BIT;
            const uint32_t word = t < 32u ? rmask : smask;
            s_off = (uint32_t)pix_off | (((word >> (t & 31u)) & 1u) << 31);
            s_koff = ((c0 + (uint32_t)krow0) * (uint32_t)HW + r * (uint32_t)W + sx) * 4u;
        }
        if constexpr (PERIODIC) {
            const uint32_t st = (uint32_t)k0 >> 4, period = fast_div(st, magic_RS, one_RS);
            uint32_t at = (st - period * (uint32_t)RS) * 16u;
            if (!FULL && k0 + 16 > kend) at = (uint32_t)RS * 16u + (k0 >= kend ? 16u : 0u);
            s_row = tab + (at + (uint32_t)krow0);
            s_koff = period * 16u * (uint32_t)HW * 4u;
        }
    }
    template <int SET, bool FULL, int J>
    __device__ __forceinline__ void row()
    {
        if constexpr (POINT) {
            const int kg = s_k0 + krow0 + J;
            if constexpr (FULL) regs[SET][J] = buf_load1(rsrc, (uint32_t)pix_off, (uint32_t)(kg * HW) * 4u);
            else if constexpr (KTAIL)
                regs[SET][J] = buf_load1(rsrc, (uint32_t)pix_off | (kg < s_kend ? 0u : kOobOffset), (uint32_t)(kg * HW) * 4u);
            else regs[SET][J] = buf_load1(rsrc, (uint32_t)pix_off, (uint32_t)(min(kg, s_kend - 1) * HW) * 4u);
        } else if constexpr (TAPMAJOR) {
            regs[SET][J] = buf_load1(rsrc, s_off, s_koff + (uint32_t)(J * HW) * 4u);
        } else if constexpr (PERIODIC) {
            const uint2 e = s_row[J];
            // bit 0 counts: the shift below drops the rest
            const uint32_t outside = MODE == GATHER_TAPS1 ? rmask >> e.x : (uint32_t)((((uint64_t)smask << 32) | rmask) >> e.x);
            regs[SET][J] = buf_load1(rsrc, ((uint32_t)pix_off + e.y) | (outside << 31), s_koff);
        } else {
            regs[SET][J] = gather<FULL>((uint32_t)(s_k0 + krow0 + J), s_kend);
        }
    }
    template <int SET, int STEP>
    __device__ __forceinline__ void step()
    {
        if constexpr (STEP == 0) activate<SET>();
        unit.template step<STEP>(regs[SET]);
    }
    __device__ __forceinline__ void write(u32x4 *stage) const
    {
        unit.write(stage + L::A_UNITS, L::B_PLANE, L::B_RUN, lds_off, krow0);
    }
    __device__ __forceinline__ bool lossy() const { return split_lossy(unit.seen); }
    template <int SET>
    __device__ __forceinline__ void store(float *Bs, int)
    {
        activate<SET>();
#pragma unroll
        for (int i = 0; i < ITERS; ++i) Bs[lds_off + i * KSTEP * T::LDB] = regs[SET][i];
    }
};

__device__ __forceinline__ float apply_act(float v, int act)
{
    if (act != POLYDL_ACT_NONE) v = fmaxf(v, 0.f);
    if (act == POLYDL_ACT_RELU6) v = fminf(v, 6.f);
    return v;
}

// Which tile, and which part of its reduction, a workgroup takes (uniform).
struct ConvPart {
    int tile, part, parts, first_split_tile, m0, n0, kbegin, kend;
};
template <class T>
__device__ __forceinline__ ConvPart conv_part(const ConvKArgs &p)
{
    ConvPart c;
    c.tile = blockIdx.x; c.part = blockIdx.y; c.parts = p.split_k; c.first_split_tile = 0;
    int kps = p.k_per_split;
    if (p.tail_parts > 1) {
        c.part = 0; c.parts = 1; c.first_split_tile = p.whole_tiles;
        if (c.tile >= p.whole_tiles) {
            uint32_t rem;
            c.tile = p.whole_tiles + (int)div_by((uint32_t)(c.tile - p.whole_tiles), (uint32_t)p.tail_parts, p.recip_tail, rem);
            c.part = (int)rem; c.parts = p.tail_parts; kps = p.tail_k;
        }
    }
    int tm, tn;
    tile_coords(c.tile, p.raster, p.tiles_m, p.tiles_n, tm, tn);
    c.m0 = tm * T::BM; c.n0 = tn * T::BN;
    c.kbegin = c.part * kps;
    c.kend = min(p.Kg, c.kbegin + kps);
    return c;
}

// What follows the reduction: the hand-over of a split reduction's parts (AHEAD of them requested together), then bias,
// activation, store.
template <class T, int AHEAD>
__device__ __forceinline__ void conv_finish(const ConvKArgs &p, const ConvPart &c, v16f (&acc)[T::MB][T::NB], int tid,
                                            int wm0, int wn0)
{
    const int lane = tid & 63, m0 = c.m0, n0 = c.n0, part = c.part, parts = c.parts;
    // With the reduction of a tile split over several workgroups every part leaves its accumulator tile in scratch
    // memory (thread-contiguous, device-scope stores); the part that arrives last adds all parts
    // in index order and runs the fused epilogue.  Nothing waits on another workgroup.
    if (parts > 1) {
        __shared__ unsigned s_arrived;
        constexpr size_t TILE = (size_t)T::BM * T::BN;
        const int slot = c.tile - c.first_split_tile;   // scratch tiles and counters are numbered over the split tiles
        float *tile0 = p.partials + (size_t)slot * parts * TILE;
        float *mine = tile0 + (size_t)part * TILE;
        store_partial_tile<T>(mine, tid, acc);
        wait_vmcnt0();   // vmcnt(0): this wave's device-scope stores have completed
        __syncthreads();
        if (tid == 0)
            s_arrived = __hip_atomic_fetch_add(p.counters + slot, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_arrived) != (unsigned)parts - 1u) return;   // not the last part
        if (tid == 0)               // leave the counter at zero for the next launch
            __hip_atomic_store(p.counters + slot, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sum_partial_tiles<T, AHEAD>(tile0, parts, tid, acc);
    }
    // epilogue.  The lane owns NB adjacent pixels starting at colg for 16*MB output channels.
    // Addresses are a per-lane byte offset from the first image the tile touches plus a uniform
    // offset per channel row, so a store costs no address arithmetic.
    const int colg = n0 + wn0 + T::NB * (lane & 31);
    if (colg >= p.Ng) return;
    const int krow = m0 + wm0 + 4 * (lane >> 5);   // channel of register 0; register r adds 8*(r/4) + r%4
    const uint32_t KPQ = (uint32_t)p.K * (uint32_t)p.PQ;
    uint32_t rem0, pq;
    const uint32_t img0 = div_by((uint32_t)n0, (uint32_t)p.PQ, p.recip_PQ, rem0);   // uniform
    const uint32_t img = div_by((uint32_t)colg, (uint32_t)p.PQ, p.recip_PQ, pq);
    const uint64_t skip = (uint64_t)img0 * KPQ * 4;
    __amdgpu_buffer_rsrc_t ro = make_rsrc(reinterpret_cast<char *>(p.out) + skip, p.out_bytes - skip);
    // bias of channels at or past K reads as zero (as does every channel without a bias vector)
    __amdgpu_buffer_rsrc_t rb = make_rsrc(p.bias, p.bias ? (uint64_t)p.K * 4 : 0);
    float bias[T::MB][16];
#pragma unroll
    for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            bias[bi][r] = buf_load1(rb, (uint32_t)(krow + 32 * bi + 8 * (r >> 2) + (r & 3)) * 4u);
    const uint32_t row_bytes = (uint32_t)p.PQ * 4u;
    // the NB pixels are one vector store when they lie in one image and keep the alignment
    const bool vec = (p.PQ % T::NB == 0) && (((uintptr_t)p.out & 15) == 0);
    if (vec) {
        const uint32_t off = ((img - img0) * KPQ + (uint32_t)krow * (uint32_t)p.PQ + pq) * 4u;
        store_rows_by<T>(p.act, m0 + T::BM <= p.K, ro, off, row_bytes, acc, bias, krow, p.K);
    } else {
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj) {
            if (colg + bj >= p.Ng) break;
            // pixel bj of the lane: same image, or among the first pixels of a following one
            uint32_t q = pq + bj, im = img - img0;
            while (q >= (uint32_t)p.PQ) { q -= (uint32_t)p.PQ; ++im; }
            const uint32_t off = (im * KPQ + (uint32_t)krow * (uint32_t)p.PQ + q) * 4u;
#pragma unroll
            for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int ch = 32 * bi + 8 * (r >> 2) + (r & 3);
                    if (krow + ch >= p.K) continue;
                    buf_store1(ro, off, (uint32_t)ch * row_bytes, apply_act(acc[bi][bj][r] + bias[bi][r], p.act));
                }
        }
    }
}

}  // namespace polydl
