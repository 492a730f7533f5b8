// Convolution of small layers as products of single waves (wave_core.hpp).  The implicit GEMM, and the ways a load finds its
// element, are those of conv_gather.hpp; here the values of a row go to LDS as they are loaded, a lane per pixel.
#include "conv_gather.hpp"
#include "wave_core.hpp"

namespace polydl {

struct ConvWaveKArgs {
    const void *in, *wt;      // float tensors, or tensors of units of eight bfloat16 channels (C counts units, Kg units of a filter row)
    const float *bias;
    float *out;
    int C, H, W, K, R, S, stride, pad;
    int PQ, Q, RS, HW, CHW, Kg, Ng;
    uint32_t magic_C, magic_RS, one_RS, magic_S, one_S;   // for fast_div()
    uint32_t recip_PQ, recip_Q;                           // for div_by()
    uint64_t in_bytes, out_bytes;
    int act, pre_act;
    WaveOrder order;
    WaveParts parts;
};

// B operand: rows of the im2col matrix.  MODE: GATHER_POINT, GATHER_TAPS1, GATHER_TAPS2 or GATHER_TAPMAJOR.  A lane loads one pixel: with
// 64 pixels a tile a row per load, with 32 two rows, the second in the upper half-wave.
template <class T, int MODE>
struct WaveBGather {
    static constexpr bool POINT = MODE == GATHER_POINT, TAPMAJOR = MODE == GATHER_TAPMAJOR;
    static constexpr bool TABLE = MODE == GATHER_TAPS1 || MODE == GATHER_TAPS2;
    static constexpr int LAST_BIT = MODE == GATHER_TAPS1 ? 31 : 63;   // never a tap: always set
    static constexpr int ROWS = 64 / T::WN, LOADS = 16 / ROWS;
    // TABLE: (tap number, byte distance) of the rows of one period of RS steps, then the last step's as it ends
    static constexpr int TABLE_ROWS = TABLE ? (LAST_BIT + 1) * 16 : 1;
    const char *base;
    uint32_t bytes;
    uint32_t pix_off, lo, hi;         // byte offset of tap (0,0), or out of range; one bit per tap, set where it lies outside the image
    int half_row;                     // ROWS == 2: the lane's row of a load
    int C, HW, W, S, RS, Kg, pre_act;
    uint32_t magic_C, magic_RS, one_RS, magic_S, one_S;
    const uint2 *tab;
    // of the step being fetched
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t off, koff;
    int k0;
    bool live;
    uint2 rows[TABLE ? LOADS : 1];

    static __device__ __forceinline__ void fill_table(const ConvWaveKArgs &p, int tid, uint2 *t)
    {
        if constexpr (TABLE) {
            const uint32_t period = (uint32_t)p.RS * 16u, last = (uint32_t)(p.Kg - 1) & ~15u;
            const uint32_t st = last >> 4, first_of_last = (st - fast_div(st, p.magic_RS, p.one_RS) * (uint32_t)p.RS) * 16u;
            for (uint32_t e = tid; e < period + 16u; e += T::THREADS) {
                const uint32_t r16 = e < period ? e : first_of_last + (e - period);
                const bool in = e < period || last + (e - period) < (uint32_t)p.Kg;
                const uint32_t c = fast_div(r16, p.magic_RS, p.one_RS), rs = r16 - c * (uint32_t)p.RS;
                const uint32_t r = fast_div(rs, p.magic_S, p.one_S), s = rs - r * (uint32_t)p.S;
                t[e] = (uint2){in ? rs : (uint32_t)LAST_BIT, (c * (uint32_t)p.HW + r * (uint32_t)p.W + s) * 4u};
            }
        }
    }
    __device__ __forceinline__ void init(const ConvWaveKArgs &p, int n0, int lane, const uint2 *t)
    {
        C = p.C; HW = p.HW; W = p.W; S = p.S; RS = p.RS; Kg = p.Kg; pre_act = p.pre_act;
        magic_C = p.magic_C; magic_RS = p.magic_RS; one_RS = p.one_RS; magic_S = p.magic_S; one_S = p.one_S;
        tab = t;
        half_row = ROWS == 2 ? lane >> 5 : 0;
        uint32_t rem0;
        const int img0 = (int)div_by((uint32_t)n0, (uint32_t)p.PQ, p.recip_PQ, rem0);
        const uint64_t skip = (uint64_t)img0 * p.CHW * 4;
        // tap (0,0) lies up to pad rows and columns before the image: the descriptor starts that much earlier
        const int lead = POINT ? 0 : (p.pad * p.W + p.pad) * 4;
        base = reinterpret_cast<const char *>(p.in) + skip - lead;
        const uint64_t left = p.in_bytes - skip + lead;
        bytes = left > kMaxRecords ? (uint32_t)kMaxRecords : (uint32_t)left;
        const int col = n0 + lane % T::WN;
        pix_off = kOobOffset;
        lo = hi = 0xFFFFFFFFu;
        if (col < p.Ng) {
            uint32_t pq, q;
            const int img = (int)div_by((uint32_t)col, (uint32_t)p.PQ, p.recip_PQ, pq), oh = (int)div_by(pq, (uint32_t)p.Q, p.recip_Q, q);
            const int ih0 = oh * p.stride - p.pad, iw0 = (int)q * p.stride - p.pad;
            pix_off = (uint32_t)(((img - img0) * p.CHW + ih0 * p.W + iw0) * 4 + lead);
            if constexpr (!POINT) {
                constexpr int MAX = MODE == GATHER_TAPS1 ? 31 : 32;
                const uint32_t rows_out = outside_bits<MAX>(-ih0, p.H - ih0, p.R), cols_out = outside_bits<MAX>(-iw0, p.W - iw0, p.S);
                const uint32_t all_cols = low_bits<MAX>(p.S);
                uint64_t taps = 0;
                for (int r = 0; r < p.R; ++r) taps |= (uint64_t)((rows_out >> r) & 1u ? all_cols : cols_out) << (r * p.S);
                lo = (uint32_t)taps;
                hi = (uint32_t)(taps >> 32);
                if constexpr (MODE == GATHER_TAPS1) lo |= 1u << 31;
                else hi |= 1u << 31;
            }
        }
        if constexpr (TABLE) {   // such a pixel's bits are all set
            if (col >= p.Ng) pix_off = 0;
        } else if constexpr (ROWS == 2) {
            if (col < p.Ng) pix_off += (uint32_t)(half_row * p.HW) * 4u;
        }
    }
    __device__ __forceinline__ void begin(int t, bool live_)
    {
        k0 = 16 * t;
        live = live_;
        rsrc = raw_rsrc(base, live ? bytes : 0u);
        if constexpr (TAPMAJOR) {   // one tap for the whole step
            const uint32_t tap = __umulhi((uint32_t)k0, magic_C), c0 = (uint32_t)k0 - tap * (uint32_t)C;
            const uint32_t r = fast_div(tap, magic_S, one_S), s = tap - r * (uint32_t)S;
            const uint32_t word = tap < 32u ? lo : hi;
            off = pix_off | (((word >> (tap & 31u)) & 1u) << 31);
            koff = (c0 * (uint32_t)HW + r * (uint32_t)W + s) * 4u;
        }
        if constexpr (TABLE) {      // the rows' entries together: one by one, each load would wait for its own
            const uint32_t period = fast_div((uint32_t)t, magic_RS, one_RS);
            const uint2 *row = tab + (k0 + 16 > Kg ? (uint32_t)RS * 16u : ((uint32_t)t - period * (uint32_t)RS) * 16u) + half_row;
#pragma unroll
            for (int n = 0; n < LOADS; ++n) rows[n] = row[n * ROWS];
            koff = period * 16u * (uint32_t)HW * 4u;
        }
    }
    template <int N>
    __device__ __forceinline__ void load(v4f *dst) const
    {
        v4f *at = dst + N * 16;
        if constexpr (POINT) {
            const int k = k0 + N * ROWS;
            if constexpr (ROWS == 1) lds_load<4>(raw_rsrc(base, live && k < Kg ? bytes : 0u), at, pix_off, (uint32_t)(k * HW) * 4u);
            else lds_load<4>(rsrc, at, k + half_row < Kg ? pix_off : kOobOffset, (uint32_t)(k * HW) * 4u);
        } else if constexpr (TAPMAJOR) {
            lds_load<4>(rsrc, at, off, koff + (uint32_t)(N * ROWS * HW) * 4u);
        } else {
            const uint2 e = rows[N];
            // bit 0 counts: the shift below drops the rest
            const uint32_t outside = MODE == GATHER_TAPS1 ? lo >> e.x : (uint32_t)((((uint64_t)hi << 32) | lo) >> e.x);
            lds_load<4>(rsrc, at, (pix_off + e.y) | (outside << 31), koff);
        }
    }
    __device__ __forceinline__ void finish(float (&v)[8]) const
    {
        if (pre_act != POLYDL_ACT_NONE) {   // uniform
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = apply_act(v[i], pre_act);
        }
    }
};

// Bias, activation and store of a lane's four channels of unit u.
template <class T>
__device__ __forceinline__ void conv_wave_store(const ConvWaveKArgs &p, int m0, int n0, int lane, int u, const v4f (&v)[T::NB])
{
    const int ch = m0 + 32 * (u / 4) + 8 * (u % 4) + 4 * (lane >> 5), col = n0 + (lane & 31);
    const uint32_t KPQ = (uint32_t)p.K * (uint32_t)p.PQ, row_bytes = (uint32_t)p.PQ * 4u;
    uint32_t rem0;
    const uint32_t img0 = div_by((uint32_t)n0, (uint32_t)p.PQ, p.recip_PQ, rem0);
    const uint64_t skip = (uint64_t)img0 * KPQ * 4;
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(reinterpret_cast<char *>(p.out) + skip, p.out_bytes - skip);
    const v4f bias = buf_load4(make_rsrc(p.bias, p.bias ? (uint64_t)p.K * 4 : 0), (uint32_t)ch * 4u);   // zero past K
#pragma unroll
    for (int bj = 0; bj < T::NB; ++bj) {
        uint32_t pq;
        const uint32_t img = div_by((uint32_t)(col + 32 * bj), (uint32_t)p.PQ, p.recip_PQ, pq);
        const uint32_t off = col + 32 * bj < p.Ng ? ((img - img0) * KPQ + (uint32_t)ch * (uint32_t)p.PQ + pq) * 4u : kOobOffset;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            buf_store1(ro, ch + e < p.K ? off : kOobOffset, e * row_bytes, apply_act(v[bj][e] + bias[e], p.act));
    }
}

template <class T, int MODE>
__global__ __launch_bounds__(T::THREADS, T::WAVES_PER_SIMD) void conv_wave_kernel(ConvWaveKArgs p)
{
    typedef WaveBGather<T, MODE> Gather;
    extern __shared__ __attribute__((aligned(16))) v4f slices[];
    __shared__ __attribute__((aligned(16))) uint2 tab[Gather::TABLE_ROWS];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    wave_tile(p.order, blockIdx.x, tm, tn);
    const int m0 = tm * T::WM, n0 = tn * T::WN;
    const int first = blockIdx.y * p.parts.part_steps, last = min(p.parts.steps, first + p.parts.part_steps);
    v16f acc[T::MB][T::NB];
    {
        WaveA<T> al;
        Gather bl;
        Gather::fill_table(p, tid, tab);
        al.init(static_cast<const float *>(p.wt), m0, p.K, p.Kg, lane);
        bl.init(p, n0, lane, tab);
        if constexpr (Gather::TABLE) __syncthreads();
        wave_products<T>(al, bl, acc, first + wave, last, p.Kg, slices + wave * T::SLICE, lane);
    }
    wave_finish<T>(slices, acc, p.parts, wave, lane, [&](int u, const v4f (&v)[T::NB]) __attribute__((always_inline)) {
        conv_wave_store<T>(p, m0, n0, lane, u, v);
    });
}

// bfloat16: a step is four reduction units of eight channels, 64 bytes of a filter row, two matrix instructions a block.  The filter goes
// through LDS as in WaveA; a pixel's unit is a lane's operand as it lies in memory, 512 consecutive bytes for a half-wave.  Four steps
// are under way.  Bound on more than a few steps: the 64 bytes a cycle a compute unit loads (8 KB a step of 64x64).  Tiles of 64x64 of
// more than one round of workgroups are shared by four waves: two workgroups on a compute unit, one loads while the other's waves meet and store
// (256 -> 484 3x3/2 on 28x28, batch 64, 73 -> 54 us, 128 -> 128 5x5/2 there 24.9 -> 20.6).
template <int MB_, int NB_, int WAVES_>
struct WaveTileBf16 {
    static constexpr int MB = MB_, NB = NB_, WAVES = WAVES_, THREADS = 64 * WAVES, WM = 32 * MB, WN = 32 * NB, UNITS = 4 * MB, DEPTH = 4;
    static constexpr int STEP = WM * 4, SUMS = UNITS * NB * 64;                            // 16-byte words
    static constexpr int SLICE = SUMS > DEPTH * STEP ? SUMS : DEPTH * STEP;
    static constexpr int LDS_BYTES = WAVES * SLICE * 16;
    static constexpr int WAVES_PER_SIMD = MB * NB == 1 ? 4 : 2;
};

// LONG: filters of 32 .. 63 taps
template <class T, bool LONG>
__global__ __launch_bounds__(T::THREADS, T::WAVES_PER_SIMD) void conv_wave_bf16_kernel(ConvWaveKArgs p)
{
    constexpr int LAST_BIT = LONG ? 63 : 31, DEPTH = T::DEPTH, A_LOADS = 2 * T::MB, LOADS = A_LOADS + 2 * T::NB;
    extern __shared__ __attribute__((aligned(16))) v4f slices[];
    __shared__ __attribute__((aligned(16))) uint2 tab[(LAST_BIT + 1) * 4];   // (tap number, byte distance) of the units of one period of RS steps, then of the last step
    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, j = lane & 31, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    wave_tile(p.order, blockIdx.x, tm, tn);
    const int m0 = tm * T::WM, n0 = tn * T::WN;
    const int first = blockIdx.y * p.parts.part_steps, last = min(p.parts.steps, first + p.parts.part_steps);
    {
        const uint32_t period = (uint32_t)p.RS * 4u, end = (uint32_t)(p.Kg - 1) & ~3u, st = end >> 2;
        const uint32_t first_of_last = (st - fast_div(st, p.magic_RS, p.one_RS) * (uint32_t)p.RS) * 4u;
        for (uint32_t e = tid; e < period + 4u; e += T::THREADS) {
            const uint32_t u = e < period ? e : first_of_last + (e - period);
            const bool in = e < period || end + (e - period) < (uint32_t)p.Kg;
            const uint32_t c = fast_div(u, p.magic_RS, p.one_RS), rs = u - c * (uint32_t)p.RS;
            const uint32_t r = fast_div(rs, p.magic_S, p.one_S), s = rs - r * (uint32_t)p.S;
            tab[e] = (uint2){in ? rs : (uint32_t)LAST_BIT, (c * (uint32_t)p.HW + r * (uint32_t)p.W + s) * 16u};
        }
    }
    WaveA<T> al;
    al.init(static_cast<const float *>(p.wt), m0, p.K, p.Kg * 4, lane);
    const int quad = (lane & 3) ^ al.turn(lane >> 2);          // the unit of a step this lane loads
    const int a_at[2] = {j * 4 + (half ^ al.turn(j)), j * 4 + ((2 + half) ^ al.turn(j))};
    uint32_t pix_off[T::NB], lo[T::NB], hi[T::NB];
    uint32_t rem0;
    const int img0 = (int)div_by((uint32_t)n0, (uint32_t)p.PQ, p.recip_PQ, rem0);
    const uint64_t skip = (uint64_t)img0 * p.CHW * 16;
    const int lead = (p.pad * p.W + p.pad) * 16;               // tap (0,0) may lie this far before the image
    const char *in = static_cast<const char *>(p.in) + skip - lead;
    const uint64_t left = p.in_bytes - skip + lead;
    const uint32_t in_bytes = left > kMaxRecords ? (uint32_t)kMaxRecords : (uint32_t)left;
#pragma unroll
    for (int bj = 0; bj < T::NB; ++bj) {
        const int col = n0 + 32 * bj + j;
        pix_off[bj] = 0;
        lo[bj] = hi[bj] = 0xFFFFFFFFu;
        if (col < p.Ng) {
            uint32_t pq, q;
            const int img = (int)div_by((uint32_t)col, (uint32_t)p.PQ, p.recip_PQ, pq), oh = (int)div_by(pq, (uint32_t)p.Q, p.recip_Q, q);
            const int ih0 = oh * p.stride - p.pad, iw0 = (int)q * p.stride - p.pad;
            pix_off[bj] = (uint32_t)(((img - img0) * p.CHW + ih0 * p.W + iw0) * 16 + lead);
            constexpr int MAX = LONG ? 32 : 31;
            const uint32_t rows_out = outside_bits<MAX>(-ih0, p.H - ih0, p.R), cols_out = outside_bits<MAX>(-iw0, p.W - iw0, p.S);
            const uint32_t all_cols = low_bits<MAX>(p.S);
            uint64_t taps = 0;
            for (int r = 0; r < p.R; ++r) taps |= (uint64_t)((rows_out >> r) & 1u ? all_cols : cols_out) << (r * p.S);
            lo[bj] = (uint32_t)taps;
            hi[bj] = (uint32_t)(taps >> 32);
            if constexpr (LONG) hi[bj] |= 1u << 31;
            else lo[bj] |= 1u << 31;
        }
    }
    __syncthreads();

    v16f acc[T::MB][T::NB];
#pragma unroll
    for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;
    v4f *slice = slices + wave * T::SLICE;
    u32x4 b[DEPTH][2][T::NB];
    auto load = [&](auto set, int t) __attribute__((always_inline)) {
        constexpr int SET = decltype(set)::value;
        const bool live = t < last;
        al.begin(t, live);
        const uint32_t behind = 4 * t + quad < p.Kg ? 0u : kOobOffset;      // a unit past the end of a filter row is the next row's first
        static_for<0, A_LOADS>([&](auto n) __attribute__((always_inline)) {
            lds_load<16>(al.rsrc, slice + SET * T::STEP + decltype(n)::value * 64, al.off[decltype(n)::value] | behind);
        });
        const uint32_t period = fast_div((uint32_t)t, p.magic_RS, p.one_RS), koff = period * 4u * (uint32_t)p.HW * 16u;
        const uint2 *row = tab + (4 * t + 4 > p.Kg ? (uint32_t)p.RS * 4u : ((uint32_t)t - period * (uint32_t)p.RS) * 4u) + half;
        const __amdgpu_buffer_rsrc_t r = raw_rsrc(in, live ? in_bytes : 0u);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint2 e = row[2 * i];
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj) {
                // bit 0 counts: the shift below drops the rest
                const uint32_t outside = LONG ? (uint32_t)((((uint64_t)hi[bj] << 32) | lo[bj]) >> e.x) : lo[bj] >> e.x;
                b[SET][i][bj] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)((pix_off[bj] + e.y) | (outside << 31)), (int)koff, 0));
            }
        }
    };
    auto multiply = [&](auto set) __attribute__((always_inline)) {
        constexpr int SET = decltype(set)::value;
        u32x4 a[2][T::MB];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int bi = 0; bi < T::MB; ++bi) a[i][bi] = __builtin_bit_cast(u32x4, slice[SET * T::STEP + bi * 128 + a_at[i]]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
                for (int bj = 0; bj < T::NB; ++bj) acc[bi][bj] = mfma_bf16(a[i][bi], b[SET][i][bj], acc[bi][bj]);
    };
    int t = first + wave;
    static_for<0, DEPTH>([&](auto n) __attribute__((always_inline)) {
        load(n, t + T::WAVES * decltype(n)::value);
        __builtin_amdgcn_sched_barrier(0);
    });
    // behind a step's filter rows come its pixels and the steps after it, which are the only ones left under way when it begins
    for (; t + T::WAVES * (DEPTH - 1) < last; t += T::WAVES * DEPTH) {
        static_for<0, DEPTH>([&](auto n) __attribute__((always_inline)) {
            __builtin_amdgcn_sched_barrier(0);
            wait_vmcnt<(DEPTH - 1) * LOADS>();
            __builtin_amdgcn_sched_barrier(0);
            multiply(n);
            __builtin_amdgcn_sched_barrier(0);
            load(n, t + T::WAVES * (DEPTH + decltype(n)::value));
        });
    }
    wait_vmcnt0();     // what was requested past the end still writes zeros into the slice
    static_for<0, DEPTH - 1>([&](auto n) __attribute__((always_inline)) {
        if (t + T::WAVES * decltype(n)::value < last) multiply(n);   // uniform
    });
    wave_finish<T>(slices, acc, p.parts, wave, lane, [&](int u, const v4f (&v)[T::NB]) __attribute__((always_inline)) {
        conv_wave_store<T>(p, m0, n0, lane, u, v);
    });
}

// rows: reduction elements of a step
template <class T>
static hipError_t conv_wave_args(const ConvProblem &q, int elem_bytes, int rows, int parts, hipStream_t stream, ConvWaveKArgs *a, int *tiles)
{
    a->in = q.in; a->wt = q.wt_tap ? q.wt_tap : q.wt;
    a->bias = q.bias; a->out = q.out;
    a->C = q.C; a->H = q.H; a->W = q.W; a->K = q.K; a->R = q.R; a->S = q.S;
    a->stride = q.stride; a->pad = q.pad; a->Q = q.Q;
    a->PQ = q.P * q.Q; a->RS = q.R * q.S; a->HW = q.H * q.W; a->CHW = q.C * q.H * q.W;
    a->Kg = q.C * a->RS; a->Ng = q.N * a->PQ;
    a->magic_C = div_magic((uint32_t)q.C);
    a->magic_RS = div_magic((uint32_t)a->RS); a->one_RS = a->RS == 1 ? 0xFFFFFFFFu : 0u;
    a->magic_S = div_magic((uint32_t)q.S); a->one_S = q.S == 1 ? 0xFFFFFFFFu : 0u;
    a->recip_PQ = div_recip((uint32_t)a->PQ); a->recip_Q = div_recip((uint32_t)q.Q);
    a->in_bytes = (uint64_t)q.N * a->CHW * elem_bytes;
    a->out_bytes = (uint64_t)q.N * q.K * a->PQ * 4;
    a->act = q.act; a->pre_act = q.pre_act;
    const int tiles_m = (q.K + T::WM - 1) / T::WM, tiles_n = (a->Ng + T::WN - 1) / T::WN;
    *tiles = tiles_m * tiles_n;
    a->order = wave_order((uint32_t)tiles_m, (uint32_t)tiles_n);
    return wave_parts((a->Kg + rows - 1) / rows, parts, *tiles, sizeof(float) * T::WM * T::WN, q.arena, stream, &a->parts);
}

template <class T>
static hipError_t conv_wave_launch_t(const ConvProblem &q, int parts, hipStream_t stream)
{
    ConvWaveKArgs a;
    int tiles;
    const hipError_t e = conv_wave_args<T>(q, 4, 16, parts, stream, &a, &tiles);
    if (e != hipSuccess) return e;
    if (q.R == 1 && q.S == 1 && q.pad == 0) return wave_launch<T, conv_wave_kernel<T, GATHER_POINT>>(tiles, a.parts.parts, stream, a);
    if (q.wt_tap) return wave_launch<T, conv_wave_kernel<T, GATHER_TAPMAJOR>>(tiles, a.parts.parts, stream, a);
    if (a.RS <= 31) return wave_launch<T, conv_wave_kernel<T, GATHER_TAPS1>>(tiles, a.parts.parts, stream, a);
    return wave_launch<T, conv_wave_kernel<T, GATHER_TAPS2>>(tiles, a.parts.parts, stream, a);
}

// 63 taps are what the mask bits hold; the images a tile touches, read and written, and its filter rows lie within 31-bit offsets.
bool conv_wave_fits(const ConvProblem &q, int tile)
{
    const int64_t RS = (int64_t)q.R * q.S;
    return (RS <= 63 || (RS == 1 && q.pad == 0)) && conv_tile_in_range(q, tile, tile) &&
           ((int64_t)q.pad * q.W + q.pad) * 4 + (tile / ((int64_t)q.P * q.Q) + 2) * q.C * q.H * q.W * 4 < kMaxOffset;
}

hipError_t conv_wave_launch(const ConvProblem &q, int tile, int waves, int parts, hipStream_t stream)
{
    if (waves == 4) return conv_wave_launch_t<WaveTile<2, 2, 4>>(q, parts, stream);
    return tile == 64 ? conv_wave_launch_t<WaveTile<2, 2, 8>>(q, parts, stream) : conv_wave_launch_t<WaveTile<1, 1, 8>>(q, parts, stream);
}

template <class T>
static hipError_t conv_wave_bf16_launch_t(const ConvProblem &q, int parts, hipStream_t stream)
{
    ConvWaveKArgs a;
    int tiles;
    const hipError_t e = conv_wave_args<T>(q, 16, 4, parts, stream, &a, &tiles);
    if (e != hipSuccess) return e;
    if (a.RS <= 31) return wave_launch<T, conv_wave_bf16_kernel<T, false>>(tiles, a.parts.parts, stream, a);
    return wave_launch<T, conv_wave_bf16_kernel<T, true>>(tiles, a.parts.parts, stream, a);
}

// q.C counts units of eight channels
bool conv_wave_bf16_fits(const ConvProblem &q, int tile)
{
    const int64_t RS = (int64_t)q.R * q.S, images = tile / ((int64_t)q.P * q.Q) + 2, units = (int64_t)q.C * RS;
    return RS <= 63 && units * RS < (1ll << 30) && images * q.K * q.P * q.Q * 4 < kMaxOffset && tile * units * 16 < kMaxOffset &&
           ((images * q.C + 4) * q.H * q.W + (int64_t)q.pad * q.W + q.pad) * 16 < kMaxOffset;
}

hipError_t conv_wave_bf16_launch(const ConvProblem &q, int tile, int waves, int parts, hipStream_t stream)
{
    if (waves == 4) return conv_wave_bf16_launch_t<WaveTileBf16<2, 2, 4>>(q, parts, stream);
    return tile == 64 ? conv_wave_bf16_launch_t<WaveTileBf16<2, 2, 8>>(q, parts, stream) : conv_wave_bf16_launch_t<WaveTileBf16<1, 1, 8>>(q, parts, stream);
}

}  // namespace polydl
