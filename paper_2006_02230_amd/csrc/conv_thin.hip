// Convolution of few input channels into at most 64 output channels (the first layer of a network): the reduction
// C*R*S is short enough for the whole split filter to stay in LDS, and every gathered input value feeds only two 32-row
// blocks of the matrix instruction.
//
// conv_split_kernel with its row table spent 14 vector instructions per matrix instruction on such a layer (3 -> 64, 7x7,
// stride 2: matrix cores busy a quarter of the time): every value gathered, split, written to LDS and read back for one
// wave's use, the filter split again by every tile, a barrier per 16 reduction rows.  Here
//   * a workgroup per compute unit splits the filter once into LDS, in the order the matrix instruction reads it, and its
//     eight waves take 64 pixels at a time (a unit) without meeting again;
//   * a lane gathers its two pixels' values straight into registers, reduction rows 16 t + 8 (lane / 32) .. + 7 of step t, and
//     splits them there into the operand of the matrix instruction: no LDS, no barrier;
//   * one step's 24 matrix instructions have the splitting of the next step's values, the loads of the step after that and
//     the filter reads dealt out between them: six vector instructions each, what is free there.
// 3 -> 64 channels 7x7/2 on 224x224, batch 32: 80 -> 62 us (batch 64: 146 -> 112); 3x3 3 -> 32 of the same, batch 32, on
// the fp32 instruction before: 35.5 -> 25 us.
// Bound: the two waves of a SIMD share its issue.  On that layer a SIMD's matrix instructions take 47 thousand cycles and its
// other vector instructions 60 thousand (10 per matrix instruction: 6 in a step, the rest by the unit and by the filter) of the
// 120 thousand that the layer lasts, at 2.0 GHz (2.4 where power allows; the products come to 0.8 PFLOP/s); then come the
// gathered loads, whose lanes touch six lines each.  Loads two steps ahead instead of one (16 more registers, a few spilled outside the loop) were 3 .. 5 % slower.
// Up to 31 reduction rows more than the layer has are multiplied (whole pairs of steps).
// Values the split cannot hold (thin_redo): a filter with one sends every unit through the fp32 instruction, from the filter in
// LDS: 3 -> 64 7x7/2 above 107 us (value by value from memory 207; the staged tiles 173), 32 -> 64 3x3 on 56x56 58 (120; 80),
// 3 -> 64 3x3 on 112x112 34 (48; 32.5).  A pixel with one sends its block of 32 pixels there: 78 (112; 74), 39.5 (70; 37.5),
// 27.5 (35; 32).
#include "conv_gather.hpp"

namespace polydl {

constexpr int kThinThreads = 512, kThinRows = 64;
struct ConvThinKArgs {
    const float *in, *wt, *bias;
    float *out;
    int C, H, W, K, R, S, stride, pad, Q, PQ, RS, HW, CHW;
    int Kg, Ng;                   // reduction length C*R*S, number of output pixels
    uint32_t magic_RS, magic_S, one_RS, one_S;   // for fast_div()
    uint32_t recip_PQ, recip_Q;   // for div_by()
    uint64_t in_bytes, out_bytes;
    int act, pre_act;
    int steps;                    // reduction steps of 16 rows, an even number
    uint32_t units, per, rem;     // 64-pixel units; a wave takes `per` of them, `rem` waves one more
    uint32_t wave_units, step_units;   // wave w's i-th unit is w * wave_units + i * step_units
};

struct ThinPixel { uint32_t off, lo, hi; };   // byte offset of tap (0,0); one bit per tap, set where it lies outside the image

struct ThinWave {
    v16f hi[2][2], lo[2][2];      // [row block][pixel block]
    u32x4 a[2][2], b[2][2][3];    // two filter planes in turn [..][row block]; pixel planes [step parity][pixel block][plane]
    float raw[2][8];              // values of the next step
    uint4 row[2];                 // two table entries, of rows whose values are loaded next, and the two behind them
    uint32_t seen[2];             // per pixel block
};

// loads the value of one row (tap number and byte distance from the table; why in this order: conv_gather.hpp)
__device__ __forceinline__ float thin_load(const ThinPixel &px, __amdgpu_buffer_rsrc_t ri, uint32_t tap, uint32_t dist)
{
    const uint64_t taps = ((uint64_t)px.hi << 32) | px.lo;
    return buf_load1(ri, (px.off + dist) | ((uint32_t)(taps >> tap) << 31));   // the shift drops the other bits
}

// One step: the products of b[S], with everything else the wave has to do meanwhile.
// at: the lane's units of this step's filter planes; tab: the lane's table rows of the step after next, whose first pair is in
// w.row[0].
template <int S>
__device__ __forceinline__ void thin_step(ThinWave &w, const ThinPixel (&px)[2], __amdgpu_buffer_rsrc_t ri, const u32x4 *at,
                                          const uint4 *tab, int pre_act)
{
    if (pre_act != POLYDL_ACT_NONE) {   // uniform
#pragma unroll
        for (int i = 0; i < 16; ++i) w.raw[i / 8][i % 8] = apply_act(w.raw[i / 8][i % 8], pre_act);
    }
    SplitUnit<8> u[2];
    u[0].seen = w.seen[0];
    u[1].seen = w.seen[1];
    __builtin_amdgcn_sched_barrier(0);
    static_for<0, 24>([&](auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value, P = i / 4, mb = i % 4 / 2, nb = i % 2;
        constexpr int PA = P < 3 ? 0 : P < 5 ? 1 : 2, PB = P < 3 ? P : P < 5 ? P - 3 : 0;
        constexpr int X = (S + PA) % 2;
        if constexpr (P == 0) w.hi[mb][nb] = mfma_bf16(w.a[X][mb], w.b[S][nb][PB], w.hi[mb][nb]);
        else w.lo[mb][nb] = mfma_bf16(w.a[X][mb], w.b[S][nb][PB], w.lo[mb][nb]);
        // the filter planes ahead of their use: the second at 12, the third at 20, the next step's first at 24
        if constexpr (i == 4 || i == 5) w.a[(S + 1) % 2][i - 4] = at[128 + 32 * (i - 4)];
        if constexpr (i == 12 || i == 13) w.a[S][i - 12] = at[256 + 32 * (i - 12)];
        if constexpr (i == 20 || i == 21) w.a[(S + 1) % 2][i - 20] = at[384 + 32 * (i - 20)];
        // split steps: pixel block i / 12, pair i % 12 / 3 of its values, phase i % 3.  The pair's registers are free
        // behind phase 0 and take the loads of the step after next in phases 1 and 2.
        constexpr int n = i / 12, pair = i % 12 / 3, phase = i % 3;
        u[n].template step<i % 12>(w.raw[n]);
        if constexpr (phase == 0) w.row[(pair + 1) % 2] = tab[pair == 3 ? (n == 0 ? 0 : 8) : pair + 1];
        if constexpr (phase == 1) w.raw[n][2 * pair] = thin_load(px[n], ri, w.row[pair % 2].x, w.row[pair % 2].y);
        if constexpr (phase == 2) w.raw[n][2 * pair + 1] = thin_load(px[n], ri, w.row[pair % 2].z, w.row[pair % 2].w);
        __builtin_amdgcn_sched_barrier(0);
    });
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) w.b[S ^ 1][n][pl] = (u32x4){u[n].p[pl][0], u[n].p[pl][1], u[n].p[pl][2], u[n].p[pl][3]};
    w.seen[0] = u[0].seen;
    w.seen[1] = u[1].seen;
}

// Pixel blocks NB0 .. NB0 + NBS - 1 on the fp32 matrix cores, for values the split cannot hold.  The two halves of the wave take
// the rows they have in the planes too.  LOSSY: the filter lies in LDS as it is, 64 values a row; otherwise its planes add up
// to it.  16 reduction rows a step, the pixels of the next one requested before this one's products.
template <bool LOSSY, int NB0, int NBS>
__device__ __forceinline__ void thin_redo(v16f (&acc)[2][2], const ThinPixel (&px)[2], __amdgpu_buffer_rsrc_t ri, const u32x4 *at0,
                                          const float *filter, const uint4 *tab0, int steps, int pre_act)
{
    float raw[2][NBS][8];
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int n = 0; n < NBS; ++n)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mb][NB0 + n][r] = 0.f;
    auto load = [&](auto set, int t) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 e = tab0[8 * t + i];
#pragma unroll
            for (int n = 0; n < NBS; ++n) {
                raw[decltype(set)::value][n][2 * i] = thin_load(px[NB0 + n], ri, e.x, e.y);
                raw[decltype(set)::value][n][2 * i + 1] = thin_load(px[NB0 + n], ri, e.z, e.w);
            }
        }
    };
    auto step = [&](auto set, int t) __attribute__((always_inline)) {
        constexpr int S = decltype(set)::value;
        load(std::integral_constant<int, S ^ 1>{}, t + 1);   // the table holds three steps more
        float a[2][8];
#pragma unroll
        for (int mb = 0; mb < 2; ++mb) {
            if constexpr (LOSSY) {
#pragma unroll
                for (int i = 0; i < 8; ++i) a[mb][i] = filter[(16 * t + i) * kThinRows + 32 * mb];
            } else {
                const u32x4 *at = at0 + t * 384 + 32 * mb;
                const u32x4 hi = at[0], mid = at[128], lo = at[256];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    auto low = [](uint32_t w) __attribute__((always_inline)) { return __builtin_bit_cast(float, w << 16); };
                    auto high = [](uint32_t w) __attribute__((always_inline)) { return __builtin_bit_cast(float, w & 0xFFFF0000u); };
                    a[mb][2 * i] = low(hi[i]) + (low(mid[i]) + low(lo[i]));
                    a[mb][2 * i + 1] = high(hi[i]) + (high(mid[i]) + high(lo[i]));
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int n = 0; n < NBS; ++n) {
                const float b = apply_act(raw[S][n][i], pre_act);
#pragma unroll
                for (int mb = 0; mb < 2; ++mb)
                    acc[mb][NB0 + n] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[mb][i], b, acc[mb][NB0 + n], 0, 0, 0);
            }
    };
    load(std::integral_constant<int, 0>{}, 0);
#pragma unroll 1
    for (int t = 0; t < steps; t += 2) {
        step(std::integral_constant<int, 0>{}, t);
        step(std::integral_constant<int, 1>{}, t + 1);
    }
}

__global__ __launch_bounds__(kThinThreads, 2) void conv_thin_kernel(ConvThinKArgs p)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 At[];    // [step][plane][half][row]
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, j = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = p.steps;
    uint2 *tab = reinterpret_cast<uint2 *>(At + steps * 384);     // (tap number, byte distance) of every row, three steps more than there are
    float *bias = reinterpret_cast<float *>(tab + (steps + 3) * 16);

    // Three octets of a filter row in flight per thread (rows need not be aligned: buffer loads only need dwords).  Value by
    // value, with a wait per octet, this took 12 us of every launch.
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wt, (uint64_t)p.K * p.Kg * 4);
    auto filter_octets = [&](auto &&use) __attribute__((always_inline)) {
        for (int idx0 = tid; idx0 < steps * 2 * kThinRows; idx0 += 3 * kThinThreads) {
            v4f raw[3][2];
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                const int idx = idx0 + n * kThinThreads, o = idx / kThinRows, k = idx % kThinRows;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    raw[n][h] = buf_load4(rw, k < p.K && 8 * o + 4 * h < p.Kg ? (uint32_t)(k * p.Kg + 8 * o + 4 * h) * 4u : kOobOffset);
            }
#pragma unroll
            for (int n = 0; n < 3; ++n) {
                const int idx = idx0 + n * kThinThreads, o = idx / kThinRows, k = idx % kThinRows;
                if (idx >= steps * 2 * kThinRows) break;
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = 8 * o + i < p.Kg ? raw[n][i / 4][i % 4] : 0.f;   // not the next row's
                use(o, k, v);
            }
        }
    };
    bool lossy = false;
    filter_octets([&](int o, int k, const float (&v)[8]) __attribute__((always_inline)) {
        SplitUnit<8> s;
        static_for<0, SplitUnit<8>::STEPS>([&](auto st) __attribute__((always_inline)) { s.template step<decltype(st)::value>(v); });
        // or an infinity, a NaN, a value that rounds to an infinity: its remainder's exponent is all ones (so may be that of
        // several remainders together, from values of 2^17 on; then the filter is only used as it is without need)
        lossy |= split_lossy(s.seen) || (s.seen & 0x7F800000u) == 0x7F800000u;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
            At[((o >> 1) * 3 + pl) * 128 + (o & 1) * 64 + k] = (u32x4){s.p[pl][0], s.p[pl][1], s.p[pl][2], s.p[pl][3]};
    });
    for (int kg = tid; kg < (steps + 3) * 16; kg += kThinThreads) {
        uint2 e = {63u, 0u};      // never a tap: always outside
        if (kg < p.Kg) {
            const uint32_t c = fast_div((uint32_t)kg, p.magic_RS, p.one_RS), rs = (uint32_t)kg - c * (uint32_t)p.RS;
            const uint32_t r = fast_div(rs, p.magic_S, p.one_S), s = rs - r * (uint32_t)p.S;
            e.x = rs;
            e.y = (c * (uint32_t)p.HW + r * (uint32_t)p.W + s) * 4u;
        }
        tab[kg] = e;
    }
    if (tid < kThinRows) bias[tid] = p.bias && tid < p.K ? p.bias[tid] : 0.f;
    lossy = __syncthreads_or(lossy);
    float *filter = reinterpret_cast<float *>(At);
    if (__builtin_expect(lossy, 0)) {   // uniform: a filter value the split cannot hold; the planes make room for the filter as it is
        filter_octets([&](int o, int k, const float (&v)[8]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 8; ++i) filter[(8 * o + i) * kThinRows + k] = v[i];
        });
        __syncthreads();
    }

    // what is left over after equal shares goes to first waves of workgroups before second ones
    const uint32_t first = (blockIdx.x * (kThinThreads / 64) + wave) * p.wave_units;
    const uint32_t extra = (uint32_t)wave * gridDim.x + blockIdx.x;
    const uint32_t count = p.per + (extra < p.rem ? 1u : 0u);
    const u32x4 *at0 = At + half * 64 + j;
    const float *filter0 = filter + half * 8 * kThinRows + j;   // the lane's values of step t: filter0[(16 t + i) * 64]
    const uint4 *tab0 = reinterpret_cast<const uint4 *>(tab + 8 * half);   // the lane's rows of step t: tab0 + 8 t
    const uint32_t KPQ = (uint32_t)p.K * (uint32_t)p.PQ;
    const int lead = (p.pad * p.W + p.pad) * 4;   // tap (0,0) may lie this far before the image
    for (uint32_t i = 0; i < count; ++i) {
        const uint32_t n0 = (i < p.per ? first + i * p.step_units : p.units - p.rem + extra) * 64u;
        uint32_t rem0;
        const uint32_t img0 = div_by(n0, (uint32_t)p.PQ, p.recip_PQ, rem0);
        const uint64_t skip = (uint64_t)img0 * p.CHW * 4;
        const __amdgpu_buffer_rsrc_t ri = make_rsrc(reinterpret_cast<const char *>(p.in) + skip - lead, p.in_bytes - skip + lead);
        ThinPixel px[2];
        uint32_t out_off[2];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
            const uint32_t col = n0 + 32u * nb + j;
            px[nb] = {0u, 0xFFFFFFFFu, 0xFFFFFFFFu};
            out_off[nb] = kOobOffset;
            if (col < (uint32_t)p.Ng) {
                uint32_t pq, q;
                const uint32_t img = div_by(col, (uint32_t)p.PQ, p.recip_PQ, pq), oh = div_by(pq, (uint32_t)p.Q, p.recip_Q, q);
                const int ih0 = (int)oh * p.stride - p.pad, iw0 = (int)q * p.stride - p.pad;
                px[nb].off = (img - img0) * (uint32_t)p.CHW * 4u + (uint32_t)((ih0 * p.W + iw0) * 4 + lead);
                out_off[nb] = ((img - img0) * KPQ + 4u * half * (uint32_t)p.PQ + pq) * 4u;
                const uint32_t rows_out = outside_bits(-ih0, p.H - ih0, p.R), cols_out = outside_bits(-iw0, p.W - iw0, p.S);
                const uint32_t all_cols = low_bits(p.S);
                uint64_t taps = 0;
                for (int r = 0; r < p.R; ++r) taps |= (uint64_t)((rows_out >> r) & 1u ? all_cols : cols_out) << (r * p.S);
                px[nb].lo = (uint32_t)taps;
                px[nb].hi = (uint32_t)(taps >> 32) | 0x80000000u;
            }
        }
        v16f acc[2][2];
        if (__builtin_expect(lossy, 0)) {   // uniform, as below
            thin_redo<true, 0, 2>(acc, px, ri, at0, filter0, tab0, steps, p.pre_act);
        } else {
            ThinWave w;
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) { w.hi[mb][nb][r] = 0.f; w.lo[mb][nb][r] = 0.f; }
            auto load_all = [&](int t) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint4 e = tab0[8 * t + i];
#pragma unroll
                    for (int nb = 0; nb < 2; ++nb) {
                        w.raw[nb][2 * i] = thin_load(px[nb], ri, e.x, e.y);
                        w.raw[nb][2 * i + 1] = thin_load(px[nb], ri, e.z, e.w);
                    }
                }
            };
            load_all(0);
            w.a[0][0] = at0[0];
            w.a[0][1] = at0[32];
            if (p.pre_act != POLYDL_ACT_NONE) {   // uniform
#pragma unroll
                for (int i = 0; i < 16; ++i) w.raw[i / 8][i % 8] = apply_act(w.raw[i / 8][i % 8], p.pre_act);
            }
#pragma unroll
            for (int n = 0; n < 2; ++n) {
                SplitUnit<8> s;
                static_for<0, SplitUnit<8>::STEPS>([&](auto st) __attribute__((always_inline)) { s.template step<decltype(st)::value>(w.raw[n]); });
                w.seen[n] = s.seen;
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) w.b[0][n][pl] = (u32x4){s.p[pl][0], s.p[pl][1], s.p[pl][2], s.p[pl][3]};
            }
            load_all(1);
            const u32x4 *at = at0;
            const uint4 *tb = tab0 + 8 * 2;
            w.row[0] = tb[0];
            // in pairs, one set of pixel planes each; what the last step prepares is never multiplied
            for (int t = 0; t < steps; t += 2) {
                thin_step<0>(w, px, ri, at, tb, p.pre_act);
                thin_step<1>(w, px, ri, at + 384, tb + 8, p.pre_act);
                at += 768;
                tb += 16;
            }
            float f[2] = {0.f, 0.f};
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int nb = 0; nb < 2; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        acc[mb][nb][r] = w.hi[mb][nb][r] + w.lo[mb][nb][r];
                        f[nb] = __builtin_fmaf(acc[mb][nb][r], 0.f, f[nb]);
                    }
            // Rare, and all of it in here and expected not to be taken: the code then lies behind the stores, not in the middle of what
            // every unit runs (3 -> 64 3x3 on 112x112, batch 32: 26.7 -> 26.3 us).
            if (__builtin_expect(__ballot(!(f[0] + f[1] == 0.f) || split_lossy(w.seen[0] | w.seen[1])) != 0, 0)) {
                bool again[2];
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) again[nb] = __ballot(!(f[nb] == 0.f) || split_lossy(w.seen[nb])) != 0;
                if (again[0] && again[1]) thin_redo<false, 0, 2>(acc, px, ri, at0, filter0, tab0, steps, p.pre_act);
                else if (again[0]) thin_redo<false, 0, 1>(acc, px, ri, at0, filter0, tab0, steps, p.pre_act);
                else if (again[1]) thin_redo<false, 1, 1>(acc, px, ri, at0, filter0, tab0, steps, p.pre_act);
            }
        }
        // bias, activation, store: the lane's channels are 32 mb + 8 (r / 4) + 4 half + r % 4; a half-wave stores 128 consecutive bytes
        const uint64_t oskip = (uint64_t)img0 * KPQ * 4;
        const __amdgpu_buffer_rsrc_t ro = make_rsrc(reinterpret_cast<char *>(p.out) + oskip, p.out_bytes - oskip);
        const uint32_t row_bytes = (uint32_t)p.PQ * 4u;
        auto store = [&](auto act, auto full) __attribute__((always_inline)) {
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f bq = *reinterpret_cast<const v4f *>(bias + 32 * mb + 8 * q + 4 * half);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int ch = 32 * mb + 8 * q + i;
                        if (!decltype(full)::value && ch + 4 * half >= p.K) continue;
#pragma unroll
                        for (int nb = 0; nb < 2; ++nb)
                            buf_store1(ro, out_off[nb], (uint32_t)ch * row_bytes, act_of<decltype(act)::value>(acc[mb][nb][4 * q + i] + bq[i]));
                    }
                }
        };
        auto by_act = [&](auto full) __attribute__((always_inline)) {
            if (p.act == POLYDL_ACT_NONE) store(std::integral_constant<int, POLYDL_ACT_NONE>{}, full);
            else if (p.act == POLYDL_ACT_RELU) store(std::integral_constant<int, POLYDL_ACT_RELU>{}, full);
            else store(std::integral_constant<int, POLYDL_ACT_RELU6>{}, full);
        };
        if (p.K == kThinRows) by_act(std::true_type{});
        else by_act(std::false_type{});
    }
}

// LDS: filter planes, row table, bias
// the last step reads ahead half a plane past the filter: the room behind it is kept
static size_t thin_lds_bytes(int steps) { return (size_t)steps * 384 * 16 + (size_t)(steps + 3) * 16 * 8 + kThinRows * 4 + 2048; }

// 64 output channels are what a wave's accumulators hold, 63 taps the mask bits, 24 steps the LDS; the images 64 pixels touch, read
// and written, lie within 31-bit offsets.
bool conv_thin_fits(const ConvProblem &q)
{
    const int64_t RS = (int64_t)q.R * q.S, PQ = (int64_t)q.P * q.Q, images = 64 / PQ + 2;
    return q.K <= kThinRows && RS <= 63 && q.C * RS <= 24 * 16 &&
           images * q.C * q.H * q.W * 4 + ((int64_t)q.pad * q.W + q.pad) * 4 < kMaxOffset && images * q.K * PQ * 4 < kMaxOffset;
}

constexpr int64_t kLastLevelCache = 256ll << 20;
static int64_t thin_bytes(const ConvProblem &q) { return (int64_t)q.N * 4 * ((int64_t)q.C * q.H * q.W + (int64_t)q.K * q.P * q.Q); }

// Where the kernel is the faster one.  Below 6 units per compute unit (of its eight waves) the picked tile is faster: 7x7 3 -> 64 stride 2
// with 980 units 18.3 us against 21.5 here, 1568: 27.9 and 22.9, 6272: 76 and 61, 16072: 194 and 146; 3x3 16 -> 64 on 56x56
// with 1274: 19.4 and 20.4, 1813: 25.3 and 21.8; 5x5 6 -> 32 with 1511: 22.4 and 20.0, 16002: 162 and 122; 3x3 3 -> 32 with
// 9016: 49 and 32.  Below 128 rows, where the picks use the fp32 instruction, the error against 64 bits falls with it (72 rows
// 1.56e-7 -> 0.58e-7).
// Reductions of up to 80 rows: the products are not all there is to win, and two things eat it.  Work of the kernel that is not
// the layer's (rows filled up to whole pairs of steps, waves without a unit in the last round of 64 pixels each; `own` is the
// rest of it): 36 rows, 56x56, 3332 units 20.7 us on the picked tile and 22.1 here (own 0.46), 27 rows on 14x14 with 2101 units
// 12.6 and 13.1 (0.43), 24 rows on 28x28 with 2401 13.6 and 15.0 (0.44); 45 rows with 4000 units 1.04 .. 1.28 times as fast (0.69).  And
// outputs beyond the last-level cache in short image rows, where the picked tiles write longer runs: 8 -> 64 3x3 on 28x28, 40903
// units 266 and 327.  Of 4685 timings of 24 .. 384 rows and 1536 .. 40000 units, operands in the cache and not, 445 were more
// than 3 % slower here, by up to 30 %; of the 3818 within these limits 88, by up to 12 % (small images of few channels), and of the
// others 256 would have been more than 3 % faster.
// 1x1 layers read their pixels in whole lines, which the staged kernel does as well: below 128 channels it is the faster
// one (64 -> 64 on 56x56 with 2401 units 17.9 us against 21.0), above it as fast with three units a wave and more
// (256 -> 64 with 1813 units 40.7 and 30.6, 3087: 60.5 and 54, 6223: 122.8 and 125).
bool conv_thin_pays(const ConvProblem &q)
{
    const int64_t Kg = (int64_t)q.C * q.R * q.S, PQ = (int64_t)q.P * q.Q, units = ((int64_t)q.N * PQ + 63) / 64, cus = compute_units();
    if (!conv_thin_fits(q) || Kg < 24 || units < 6 * cus) return false;
    if (Kg <= 80) {
        const int64_t waves = cus * (kThinThreads / 64), rounds = (units + waves - 1) / waves, rows = (Kg + 31) / 32 * 32;
        const double own = (double)(Kg * units) / (double)(rows * rounds * waves);
        if (own < (Kg <= 48 ? 0.55 : 0.45)) return false;
        if (q.K > 32 && q.Q < 48 && thin_bytes(q) > kLastLevelCache) return false;
    }
    return q.R * q.S != 1 || (Kg >= 128 && units <= 16 * cus);
}

// Whether a wave takes its units in a run: where a unit reads at least half of its input rows again that the one before it
// read (64 pixels go 64 * stride / Q rows further, R - stride rows stay) and the layer fits the last-level cache.  There it finds
// them close by: 3 -> 64 3x3 on 112x112, 5096 units, 23.7 us against 26.2, 7x7/2 on 224x224 51.9 and 53.4.  Otherwise
// neighbouring waves take neighbouring units, so that what the card reads and writes at a time lies together: 8 -> 64 3x3/2 on
// 14x28, 9001 units, 96.0 us against 108.8 in runs, 3 -> 64 3x3 on 112x112, 25088 units, 106 and 125.5.
static bool thin_in_runs(const ConvProblem &q)
{
    return (int64_t)(q.R - q.stride) * q.Q >= 64ll * q.stride && thin_bytes(q) <= kLastLevelCache;
}

hipError_t conv_thin_launch(const ConvProblem &q, hipStream_t stream)
{
    ConvThinKArgs a;
    a.in = static_cast<const float *>(q.in); a.wt = static_cast<const float *>(q.wt);
    a.bias = q.bias; a.out = q.out;
    a.C = q.C; a.H = q.H; a.W = q.W; a.K = q.K; a.R = q.R; a.S = q.S;
    a.stride = q.stride; a.pad = q.pad; a.Q = q.Q;
    a.PQ = q.P * q.Q; a.RS = q.R * q.S; a.HW = q.H * q.W; a.CHW = q.C * q.H * q.W;
    a.Kg = q.C * a.RS; a.Ng = q.N * a.PQ;
    a.magic_RS = div_magic((uint32_t)a.RS); a.one_RS = a.RS == 1 ? 0xFFFFFFFFu : 0u;
    a.magic_S = div_magic((uint32_t)q.S); a.one_S = q.S == 1 ? 0xFFFFFFFFu : 0u;
    a.recip_PQ = div_recip((uint32_t)a.PQ); a.recip_Q = div_recip((uint32_t)q.Q);
    a.in_bytes = (uint64_t)q.N * a.CHW * 4;
    a.out_bytes = (uint64_t)q.N * q.K * a.PQ * 4;
    a.act = q.act; a.pre_act = q.pre_act;
    a.steps = (a.Kg + 31) / 32 * 2;
    a.units = ((uint32_t)a.Ng + 63u) / 64u;
    const uint32_t waves_per_wg = kThinThreads / 64, need = (a.units + waves_per_wg - 1) / waves_per_wg;
    const uint32_t cus = (uint32_t)compute_units(), wgs = need < cus ? need : cus, waves = wgs * waves_per_wg;
    a.per = a.units / waves;
    a.rem = a.units % waves;
    const bool runs = thin_in_runs(q);
    a.wave_units = runs ? a.per : 1;
    a.step_units = runs ? 1 : waves;
    const size_t lds = thin_lds_bytes(a.steps);
    if (lds > 64 * 1024) {   // more than the default window has to be asked for
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(conv_thin_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)thin_lds_bytes(24));
        if (e != hipSuccess) return e;
    }
    return launch_kernel(conv_thin_kernel, dim3(wgs), dim3(kThinThreads), lds, stream, a);
}

}  // namespace polydl
