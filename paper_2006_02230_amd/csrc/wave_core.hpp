// Small products on split operands (split_core.hpp), without stages that waves share: a wave brings its own operands, splits
// them in registers and multiplies.  The waves of a workgroup (eight, or four) work on one tile of the result and take the reduction's
// steps of 16 rows in turn; they meet once, at the end, in LDS.  No barrier in the loop, no trip through scratch memory
// unless a tile's reduction is dealt to several workgroups.
//
// The staged kernels pay a barrier, an LDS round trip and a wait for every 16 rows and a hand-over through memory for every part of
// a reduction that eight workgroups share; on a problem of a few stages per workgroup that is most of its time.  Here every wave
// splits its operands for itself, 192 vector instructions per 24 matrix instructions with 64x64 tiles (the staged 128x128 tile: 96),
// so large problems stay with the staged kernels.  Bound: those vector instructions beside the products.  Two waves of a SIMD take
// 2710 cycles for a step of 64x64x16 each, 1536 of matrix cores; the bare splitting and products, no loads, take 2430.
#pragma once
#include <atomic>

#include "gemm_core.hpp"
#include "internal.hpp"
#include "split_core.hpp"

namespace polydl {

// Tile of MB x NB blocks of 32 x 32, shared by WAVES waves.
template <int MB_, int NB_, int WAVES_>
struct WaveTile {
    static constexpr int MB = MB_, NB = NB_, WAVES = WAVES_, THREADS = 64 * WAVES, WM = 32 * MB, WN = 32 * NB;
    static constexpr int UNITS = 4 * MB;                       // (row block, register quad) of the accumulators
    static constexpr int A_WORDS = WM * 4, B_WORDS = WN * 4;   // 16-byte words of a step's operands in LDS
    static constexpr int STEP = A_WORDS + B_WORDS;
    static constexpr int SUMS = UNITS * NB * 64;               // and of a wave's accumulators
    static constexpr int SLICE = SUMS > 2 * STEP ? SUMS : 2 * STEP;   // a wave's own part of LDS: two steps, later its sums
    static constexpr int LDS_BYTES = WAVES * SLICE * 16;
    static constexpr int WAVES_PER_SIMD = MB * NB == 1 ? 4 : 2;
};

// Which tile a workgroup takes: the order of tile_coords(), raster 1, without its divisions.
struct WaveOrder {
    uint32_t per, rem;                    // tiles of an XCD, of how many one more
    uint32_t band, recip_band;            // tiles of eight tile rows
    uint32_t bands, last_rows, recip_last;   // whole bands, tile rows of what is left
};
inline WaveOrder wave_order(uint32_t tiles_m, uint32_t tiles_n)
{
    WaveOrder o;
    const uint32_t total = tiles_m * tiles_n;
    o.per = total / 8; o.rem = total % 8;
    o.band = 8 * tiles_n; o.recip_band = div_recip(o.band);
    o.bands = tiles_m / 8; o.last_rows = tiles_m % 8;
    o.recip_last = div_recip(o.last_rows ? o.last_rows : 1);
    return o;
}
__device__ __forceinline__ void wave_tile(const WaveOrder &o, uint32_t pid, int &tm, int &tn)
{
    const uint32_t x = pid & 7, seq = x * o.per + min(x, o.rem) + (pid >> 3);
    uint32_t in_band, r;
    const uint32_t g = div_by(seq, o.band, o.recip_band, in_band);
    if (g < o.bands) { tn = (int)(in_band >> 3); r = in_band & 7; }
    else tn = (int)div_by(in_band, o.last_rows, o.recip_last, r);
    tm = (int)(8 * g + r);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, 0x00020000);
}

// waits until at most N of the wave's vector-memory operations are still under way (encoding: wait_vmcnt0())
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | (N >> 4 << 14) | 0x0F70);
}

// lane i's BYTES bytes to dst + i * BYTES
template <int BYTES>
__device__ __forceinline__ void lds_load(__amdgpu_buffer_rsrc_t r, v4f *dst, uint32_t off, uint32_t uniform_off = 0)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (BYTES == 16) __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 16, (int)off, (int)uniform_off, 0, 0);
    else __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)dst, 4, (int)off, (int)uniform_off, 0, 0);
#endif
}

// A operand: row-major, reduction contiguous; rows of any length and base (buffer loads need dwords only).  Lane i of the n-th load
// brings 16 bytes of row 16 n + i / 4, so that four lanes read 64 bytes of a row together (a lane's row for itself: 15 % slower
// on 1024^3); the four words of a row are swapped by its number, so that the lanes that read, each its row's eight
// values, do not meet in the same banks.
template <class T>
struct WaveA {
    static constexpr int LOADS = 2 * T::MB;
    const char *base;
    uint32_t bytes;                   // of the rows that exist from the tile's first on, at most WM
    uint32_t off[LOADS];
    int at0, at1;
    __amdgpu_buffer_rsrc_t rsrc;      // of the step being fetched
    static __device__ __forceinline__ int turn(int row) { return ((row >> 1) & 2) | (((row >> 3) ^ (row >> 1)) & 1); }
    __device__ __forceinline__ void init(const float *A, int m0, int M, int K, int lane)
    {
        const uint32_t row_bytes = (uint32_t)K * 4u;
        base = reinterpret_cast<const char *>(A) + (uint64_t)(uint32_t)m0 * row_bytes;
        bytes = (uint32_t)min(M - m0, T::WM) * row_bytes;
#pragma unroll
        for (int n = 0; n < LOADS; ++n) {
            const int row = 16 * n + (lane >> 2);
            off[n] = m0 + row < M ? (uint32_t)row * row_bytes + 16u * ((lane & 3) ^ turn(row)) : kOobOffset;
        }
        const int j = lane & 31, q = 2 * (lane >> 5);
        at0 = j * 4 + (q ^ turn(j));
        at1 = j * 4 + ((q + 1) ^ turn(j));
    }
    // live: the step exists (uniform); nothing is read otherwise
    __device__ __forceinline__ void begin(int t, bool live)
    {
        const uint32_t k = live ? 64u * (uint32_t)t : bytes;
        rsrc = raw_rsrc(base + k, bytes - k);
    }
    template <int N>
    __device__ __forceinline__ void load(v4f *dst) const { lds_load<16>(rsrc, dst + N * 64, off[N]); }
    template <int BI>
    __device__ __forceinline__ void fetch(const v4f *src, float (&v)[8]) const
    {
        const v4f x = src[BI * 128 + at0], y = src[BI * 128 + at1];
#pragma unroll
        for (int e = 0; e < 4; ++e) { v[e] = x[e]; v[4 + e] = y[e]; }
    }
};

template <class T>
struct WaveOperands {
    u32x4 a[3][T::MB], b[3][T::NB];
    uint32_t seen = 0;
    template <int N>
    __device__ __forceinline__ void put(u32x4 (&x)[3][N], int block, const float (&v)[8])
    {
        SplitUnit<8> u;
        u.seen = seen;
        static_for<0, SplitUnit<8>::STEPS>([&](auto st) __attribute__((always_inline)) { u.template step<decltype(st)::value>(v); });
        seen = u.seen;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) x[pl][block] = (u32x4){u.p[pl][0], u.p[pl][1], u.p[pl][2], u.p[pl][3]};
    }
    // the I-th product of a step
    template <int I>
    __device__ __forceinline__ void product(SplitAcc<T> &s) const
    {
        constexpr int BLOCKS = T::MB * T::NB, P = I / BLOCKS, bi = I % BLOCKS / T::NB, bj = I % T::NB;
        constexpr int PA = P == 1 || P == 3 ? 1 : P == 4 ? 2 : 0, PB = P == 2 || P == 3 ? 1 : P == 5 ? 2 : 0;
        if constexpr (P == 0) s.hi[bi][bj] = mfma_bf16(a[PA][bi], b[PB][bj], s.hi[bi][bj]);
        else s.lo[bi][bj] = mfma_bf16(a[PA][bi], b[PB][bj], s.lo[bi][bj]);
    }
};

// Steps t, t + WAVES, ... below last.  A step's values are split, then multiplied; between its products the wave requests the step
// after the next one, into the part of LDS these values came from, and reads the next one's values.  (With a descriptor per load,
// and requests and reads ahead of the splitting, 1024^3 took 18.8 us instead of 17.8, 2048^3 135 instead of 125, 512 -> 512 3x3 on 7x7, batch
// 32, 78 instead of 76; with those descriptors gone the order makes no difference.)
// The loaders' BL: begin(t, live) and load<N>(dst), N < LOADS, fill the [16][WN] image of a step, zeros for rows past the reduction's
// end (a row of A goes on with the next row's values there) and nothing where the step does not exist; finish(v) ends a block's values.
template <class T, class BL>
__device__ __forceinline__ uint32_t wave_mainloop(WaveA<T> &al, BL &bl, SplitAcc<T> &sum, int t, int last, v4f *slice, int lane)
{
    constexpr int A_LOADS = WaveA<T>::LOADS, LOADS = A_LOADS + BL::LOADS;
    constexpr int MM = 6 * T::MB * T::NB, LEAD = MM / 12, SPAN = MM * 3 / 4 - LEAD, FETCH = MM * 3 / 4;   // where requests and reads stand
    const float *b_at = reinterpret_cast<const float *>(slice + T::A_WORDS) + (lane >> 5) * 8 * T::WN + (lane & 31);
    WaveOperands<T> w;
    float va[T::MB][8], vb[T::NB][8];
    auto begin = [&](int t) __attribute__((always_inline)) {
        al.begin(t, t < last);
        bl.begin(t, t < last);
    };
    auto load = [&](auto n, int buf) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value;
        v4f *dst = slice + buf * T::STEP;
        if constexpr (N < A_LOADS) al.template load<N>(dst);
        else bl.template load<N - A_LOADS>(dst + T::A_WORDS);
    };
    // the values of the step in `buf`, of which at most the other step's loads may be under way
    auto fetch = [&](int buf) __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        wait_vmcnt<LOADS>();
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
            for (int i = 0; i < 8; ++i) vb[bj][i] = b_at[buf * T::STEP * 4 + i * T::WN + 32 * bj];
        static_for<0, T::MB>([&](auto b) __attribute__((always_inline)) { al.template fetch<decltype(b)::value>(slice + buf * T::STEP, va[decltype(b)::value]); });
        __builtin_amdgcn_sched_barrier(0);
    };
    auto step = [&](int t, auto bufc) __attribute__((always_inline)) {
        constexpr int buf = decltype(bufc)::value;
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj) {
            bl.finish(vb[bj]);
            w.put(w.b, bj, vb[bj]);
        }
#pragma unroll
        for (int bi = 0; bi < T::MB; ++bi) w.put(w.a, bi, va[bi]);
        __builtin_amdgcn_sched_barrier(0);   // the step's values are in registers: its part of LDS is free
        begin(t + 2 * T::WAVES);
        __builtin_amdgcn_sched_barrier(0);
        static_for<0, MM>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            w.template product<i>(sum);
            __builtin_amdgcn_sched_barrier(0);
            static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) {
                if constexpr (LEAD + decltype(n)::value * SPAN / LOADS == i) load(n, buf);
            });
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i == FETCH) fetch(buf ^ 1);
        });
    };
    begin(t);
    static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) { load(n, 0); });
    __builtin_amdgcn_sched_barrier(0);
    begin(t + T::WAVES);
    static_for<0, LOADS>([&](auto n) __attribute__((always_inline)) { load(n, 1); });
    fetch(0);
    // in pairs, both unconditional; an odd last one behind them (why: gemm_core.hpp)
    for (; t + T::WAVES < last; t += 2 * T::WAVES) {
        step(t, std::integral_constant<int, 0>{});
        step(t + T::WAVES, std::integral_constant<int, 1>{});
    }
    if (t < last) step(t, std::integral_constant<int, 0>{});
    wait_vmcnt0();     // what was requested past the end still writes zeros into the slice
    return w.seen;
}

// The same steps on the fp32 matrix cores, for values the split cannot hold.  K: length of the reduction.
template <class T, class BL>
__device__ __forceinline__ void wave_redo(WaveA<T> &al, BL &bl, v16f (&acc)[T::MB][T::NB], int t, int last, int K, v4f *slice, int lane)
{
    const float *src = reinterpret_cast<const float *>(slice + T::A_WORDS) + (lane >> 5) * 8 * T::WN + (lane & 31);
#pragma unroll
    for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;
#pragma unroll 1   // a step's values have been read before the next one's arrive
    for (; t < last; t += T::WAVES) {
        al.begin(t, true);
        static_for<0, WaveA<T>::LOADS>([&](auto n) __attribute__((always_inline)) { al.template load<decltype(n)::value>(slice); });
        bl.begin(t, true);
        static_for<0, BL::LOADS>([&](auto n) __attribute__((always_inline)) { bl.template load<decltype(n)::value>(slice + T::A_WORDS); });
        wait_vmcnt0();
        float a[T::MB][8], b[T::NB][8];
        static_for<0, T::MB>([&](auto n) __attribute__((always_inline)) { al.template fetch<decltype(n)::value>(slice, a[decltype(n)::value]); });
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj) {
#pragma unroll
            for (int i = 0; i < 8; ++i) b[bj][i] = src[i * T::WN + 32 * bj];
            bl.finish(b[bj]);
        }
        const int rem = K - t * 16 - 8 * (lane >> 5);   // a row's values past its end are the next row's
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
                for (int bj = 0; bj < T::NB; ++bj)
                    acc[bi][bj] = __builtin_amdgcn_mfma_f32_32x32x2f32(i < rem ? a[bi][i] : 0.f, b[bj][i], acc[bi][bj], 0, 0, 0);
    }
}

// The products of one wave: sums of its steps first + wave, + WAVES, ...
template <class T, class BL>
__device__ __forceinline__ void wave_products(WaveA<T> &al, BL &bl, v16f (&acc)[T::MB][T::NB], int t, int last, int K, v4f *slice, int lane)
{
    SplitAcc<T> sum;
    sum.clear();
    const uint32_t seen = wave_mainloop<T>(al, bl, sum, t, last, slice, lane);
    const bool bad = sum.finish(acc) || split_lossy(seen);
    if (__builtin_expect(__ballot(bad) != 0, 0)) wave_redo<T>(al, bl, acc, t, last, K, slice, lane);
}

struct WaveParts {
    int steps, part_steps, parts;    // of a tile's reduction; parts: workgroups that share it (blockIdx.y)
    float *partials;                 // parts > 1: [tile][part][SUMS] sums in register order
    unsigned *counters;              // parts > 1: per tile, how many of its parts have finished
};

// Cuts a reduction of `steps` steps, and fetches scratch memory for the parts (tiles: of the result, sums: bytes of one).
inline hipError_t wave_parts(int steps, int parts, int tiles, size_t tile_bytes, const ScratchArena *arena, hipStream_t stream, WaveParts *w)
{
    w->steps = steps;
    if (parts > w->steps) parts = w->steps;
    if (parts < 1) parts = 1;
    w->part_steps = (w->steps + parts - 1) / parts;
    w->parts = (w->steps + w->part_steps - 1) / w->part_steps;
    w->partials = nullptr;
    w->counters = nullptr;
    if (w->parts <= 1) return hipSuccess;
    return splitk_scratch(stream, arena, (size_t)tiles * w->parts * tile_bytes, tiles, &w->partials, &w->counters);
}

// A kernel that needs more than the default window of LDS has to ask for it: all of these do, the smallest with 64 KB beside its table.
// Asked once per device (threads that ask at the same time ask for the same): on every call it was 0.05 us of 3.3 on the host.
template <class T, auto KERNEL, class... A>
inline hipError_t wave_launch(int tiles, int parts, hipStream_t stream, A... args)
{
    static_assert(T::LDS_BYTES >= 64 * 1024, "with the kernel's own arrays more than the default window");
    static std::atomic<uint64_t> asked{0};   // one bit a device
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0;
    if (!(asked.load(std::memory_order_relaxed) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, T::LDS_BYTES);
        if (e != hipSuccess) return e;
        asked.fetch_or(bit, std::memory_order_relaxed);
    }
    return launch_kernel(KERNEL, dim3((unsigned)tiles, (unsigned)parts), dim3(T::THREADS), T::LDS_BYTES, stream, args...);
}

// The waves' sums meet in LDS, those of several workgroups in scratch memory (as in conv_finish()); each is added up in a
// fixed order, the same for every order of arrival.  store(u, v): the lane's four rows of unit u in every column block, called by one wave for each unit.
template <class T, class F>
__device__ __forceinline__ void wave_finish(v4f *slices, const v16f (&acc)[T::MB][T::NB], const WaveParts &p, int wave, int lane, F &&store)
{
    v4f *mine = slices + wave * T::SLICE + lane;
#pragma unroll
    for (int u = 0; u < T::UNITS; ++u)
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj) {
            const v16f &r = acc[u / 4][bj];
            mine[(u * T::NB + bj) * 64] = (v4f){r[4 * (u % 4)], r[4 * (u % 4) + 1], r[4 * (u % 4) + 2], r[4 * (u % 4) + 3]};
        }
    __syncthreads();
    // a wave's units: wave, wave + WAVES, ...; a tile of fewer units than waves leaves some without
    constexpr int MINE = (T::UNITS + T::WAVES - 1) / T::WAVES;
    static_assert(MINE == 1 || T::UNITS % T::WAVES == 0, "all waves as many units");
    const bool any = wave < T::UNITS;   // uniform
    v4f v[MINE][T::NB];
#pragma unroll
    for (int m = 0; m < MINE; ++m)
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj) {
            v[m][bj] = (v4f){0.f, 0.f, 0.f, 0.f};
            if (!any) continue;
            // in pairs: few roundings deep, so that no sum is further off than that of a staged tile's few parts
            v4f x[T::WAVES];
#pragma unroll
            for (int i = 0; i < T::WAVES; ++i) x[i] = slices[i * T::SLICE + ((wave + m * T::WAVES) * T::NB + bj) * 64 + lane];
#pragma unroll
            for (int d = 1; d < T::WAVES; d *= 2)
#pragma unroll
                for (int i = 0; i < T::WAVES; i += 2 * d) x[i] += x[i + d];
            v[m][bj] = x[0];
        }
    if (p.parts > 1) {
        __shared__ unsigned s_arrived;
        constexpr uint32_t BYTES = T::SUMS * 16;
        const char *part0 = reinterpret_cast<const char *>(p.partials) + (size_t)blockIdx.x * p.parts * BYTES;
        const int off = 16 * lane + wave * T::NB * 1024;
        if (any) {
            const __amdgpu_buffer_rsrc_t r = raw_rsrc(part0 + (size_t)blockIdx.y * BYTES, BYTES);
#pragma unroll
            for (int m = 0; m < MINE; ++m)
#pragma unroll
                for (int bj = 0; bj < T::NB; ++bj)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4i, v[m][bj]), r, off + (m * T::WAVES * T::NB + bj) * 1024, 0, kDeviceScope);
        }
        wait_vmcnt0();
        __syncthreads();
        if (threadIdx.x == 0)
            s_arrived = __hip_atomic_fetch_add(p.counters + blockIdx.x, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(s_arrived) != (unsigned)p.parts - 1u) return;   // not the last part
        if (threadIdx.x == 0) __hip_atomic_store(p.counters + blockIdx.x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (!any) return;
#pragma unroll
        for (int m = 0; m < MINE; ++m)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj) v[m][bj] = (v4f){0.f, 0.f, 0.f, 0.f};
        constexpr int AHEAD = 4;
        for (int q = 0; q < p.parts; q += AHEAD) {
            const __amdgpu_buffer_rsrc_t r = raw_rsrc(part0 + (size_t)q * BYTES, AHEAD * BYTES);
            v4f x[AHEAD][MINE][T::NB];
#pragma unroll
            for (int n = 0; n < AHEAD; ++n)
#pragma unroll
                for (int m = 0; m < MINE; ++m)
#pragma unroll
                    for (int bj = 0; bj < T::NB; ++bj)   // parts past the last one are out of range: no access, zeros
                        x[n][m][bj] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                                          r, q + n < p.parts ? off + (m * T::WAVES * T::NB + bj) * 1024 : (int)kOobOffset, n * (int)BYTES, kDeviceScope));
#pragma unroll
            for (int m = 0; m < MINE; ++m)
#pragma unroll
                for (int bj = 0; bj < T::NB; ++bj) v[m][bj] += (x[0][m][bj] + x[1][m][bj]) + (x[2][m][bj] + x[3][m][bj]);
        }
    }
    if (!any) return;
#pragma unroll
    for (int m = 0; m < MINE; ++m) store(wave + m * T::WAVES, v[m]);
}

}  // namespace polydl
