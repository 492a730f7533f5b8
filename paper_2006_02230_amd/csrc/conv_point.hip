// Pointwise convolution (R = S = 1, stride 1, no padding) with few input channels: the loop nest
// of figure "The 2-D Convolution code" (section "Convolutions") degenerates to
//   out[n][k][x] = sum_c wt[k][c] * in[n][c][x],   x = 0 .. H*W-1,
// a GEMM whose reduction (C <= 64) is so short that staging pixels through LDS, a barrier per
// stage and a tile prologue per workgroup cost more than the arithmetic.  Here
//   * the whole filter matrix sits in LDS for the life of the workgroup, split once into the three bfloat16
//     parts of split_core.hpp (K*C*6 <= 96 KB) in the order the matrix instruction reads it;
//   * a wave owns 64 pixels at a time and loads their C channels from global memory straight into
//     registers -- lane j of each half-wave holds pixels 2j and 2j+1 (one 8-byte load per channel), the
//     half-waves hold channels 0-7 and 8-15 of every 16 -- where they are split once for all channel groups;
//   * with those registers it produces the output channels in groups of 32 (accumulators: two
//     blocks of 32x32, one per pixel of the lane's pair), bias and activation applied on the way out
//     (section "Operator Fusion"), each lane storing its two pixels of a channel row as one 8-byte store;
//   * (pixel tile, channel group) units are dealt to the waves of a grid that fits the chip once
//     in contiguous, equal runs, so a wave reloads pixels only when its run crosses a tile.
// No barrier after the filter is in LDS; waves never wait for each other.
//
// Bound: the bytes written.  With the fp32 instruction the matrix cores needed 21 us of 40 for 64 -> 256 channels
// at 56x56, batch 32, and hardly overlapped with the stores; the split products need 8: 40 -> 32 us back to
// back on the same tensors (44.9 -> 37.8 with operands and outputs that are not in the caches), batch 64 69 -> 58.
#include <hip/hip_runtime.h>
#include "gemm_core.hpp"
#include "internal.hpp"
#include "split_core.hpp"

namespace polydl {

struct ConvPointKArgs {
    const float *in, *wt, *bias;
    float *out;
    int N, C, K, HW;
    int groups;             // K / 32
    uint32_t units;         // pixel tiles * groups
    uint32_t per, rem;      // units per wave; the first rem waves take one more
    uint32_t recip_groups, recip_HW;
    int act;
};

__device__ __forceinline__ v2f buf_load2(__amdgpu_buffer_rsrc_t r, uint32_t byte_off, uint32_t uniform_off)
{
    typedef int v2i __attribute__((ext_vector_type(2)));
    v2i v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)byte_off, (int)uniform_off, 0);
    return __builtin_bit_cast(v2f, v);
}

// What a finished unit leaves behind until it is stored: its two blocks of sums, bias added, the
// lane's output offset and the group's first channel.
struct PointUnit {
    v16f acc[2];
    uint32_t vo;
    int k0;
};

// Stores first .. first + count - 1 (of 16) of a finished unit: accumulator registers 4q .. 4q+3 are
// four consecutive channels, the lane's two pixels of a channel row go out as one 8-byte store.
// Called from fully unrolled loops only, so every index is a constant.
template <int ACT>
__device__ __forceinline__ void point_store(__amdgpu_buffer_rsrc_t ro, uint32_t row_bytes, const PointUnit &u,
                                            int first, int count)
{
#pragma unroll
    for (int r = first; r < first + count; ++r) {
        const int q = r >> 2, i = r & 3;
        v2f v = {act_of<ACT>(u.acc[0][r]), act_of<ACT>(u.acc[1][r])};
        buf_store2(ro, u.vo, (uint32_t)(u.k0 + 8 * q + i) * row_bytes, v);
    }
}

// The pixels of a tile, split: [pixel of the pair][block of 16 channels][part].
template <int KB>
struct PointPixels {
    u32x4 b[2][KB][3];
    uint32_t seen[2];      // SplitUnit::seen of the lane's channels of each pixel
};

// The products of one unit into `cur` and, PENDING, the 16 stores of the unit finished before it
// (`old`) dealt out between them: a wave's stores leave while its own next matrix instructions run
// instead of after them, in a phase of their own in which the matrix core of the SIMD has nothing to do
// unless another wave happens to be out of step.  True if a sum is not finite.
template <int KB, int ACT, bool PENDING>
__device__ __forceinline__ bool point_unit(const u32x4 *a_base, int K, const PointPixels<KB> &px, const v4f (&bias)[4],
                                           PointUnit &cur, __amdgpu_buffer_rsrc_t ro, uint32_t row_bytes, const PointUnit &old)
{
    v16f hi[2], lo[2];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) { hi[nb][r] = 0.f; lo[nb][r] = 0.f; }
    constexpr int PER = 16 / KB;   // stores per block of 16 channels
    static_for<0, KB>([&](auto kc) __attribute__((always_inline)) {
        constexpr int kb = decltype(kc)::value;
        u32x4 a[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) a[pl] = a_base[(kb * 3 + pl) * 2 * K];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) hi[nb] = mfma_bf16(a[0], px.b[nb][kb][0], hi[nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) lo[nb] = mfma_bf16(a[1], px.b[nb][kb][0], lo[nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) lo[nb] = mfma_bf16(a[0], px.b[nb][kb][1], lo[nb]);
        if constexpr (PENDING) {
            point_store<ACT>(ro, row_bytes, old, kb * PER, PER / 2);
            // keep the stores where they are: left alone, the scheduler moves them all behind the
            // last matrix instruction
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) lo[nb] = mfma_bf16(a[1], px.b[nb][kb][1], lo[nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) lo[nb] = mfma_bf16(a[2], px.b[nb][kb][0], lo[nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) lo[nb] = mfma_bf16(a[0], px.b[nb][kb][2], lo[nb]);
        if constexpr (PENDING) {
            point_store<ACT>(ro, row_bytes, old, kb * PER + PER / 2, PER / 2);
            __builtin_amdgcn_sched_barrier(0);
        }
    });
    float f = 0.f;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float v = hi[nb][r] + lo[nb][r];
            f = __builtin_fmaf(v, 0.f, f);
            cur.acc[nb][r] = v + bias[r >> 2][r & 3];
        }
    return !(f == 0.f);
}

// A wave's run of units [u, end).  Two unit records take turns: while one collects the products of
// unit i, the other, holding unit i - 1, is stored.
template <int KB, int ACT>
__device__ __forceinline__ void point_run(const ConvPointKArgs &p, const u32x4 *At, bool lossy_filter, uint32_t u, uint32_t end,
                                          int half, int j)
{
    const int K = p.K, C = KB * 16;
    const uint32_t HW = p.HW, total = (uint32_t)p.N * HW;
    const __amdgpu_buffer_rsrc_t ri = make_rsrc(p.in, (uint64_t)total * C * 4);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(p.out, (uint64_t)total * K * 4);
    const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.bias, p.bias ? (uint64_t)K * 4 : 0);
    const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wt, (uint64_t)K * C * 4);
    const uint32_t row_bytes = HW * 4u;

    uint32_t g;
    uint32_t tile = div_by(u, (uint32_t)p.groups, p.recip_groups, g);
    uint32_t have = 0xFFFFFFFFu, vo = kOobOffset, vi0 = kOobOffset;   // vi0: channel 0 of the lane's pixels
    PointPixels<KB> px;
    v4f bias[4];
    // pixels of a new tile, the unit's output offset and channel group, the lane's 16 bias values (zeros
    // without a bias; they are needed only when the unit's sums are complete)
    auto open_unit = [&](PointUnit &cur) {
        if (tile != have) {
            // the lane's two pixels: 2j and 2j+1 of the tile, in one image since H*W is even
            const uint32_t pix0 = tile * 64u + 2u * j;
            uint32_t x;
            const uint32_t n = div_by(pix0, HW, p.recip_HW, x);
            const bool ok = pix0 < total;
            vi0 = ok ? (n * C * HW + x) * 4u : kOobOffset;
            const uint32_t vi = ok ? vi0 + (uint32_t)(8 * half) * row_bytes : kOobOffset;
            vo = ok ? ((n * K + 4u * half) * HW + x) * 4u : kOobOffset;
            px.seen[0] = 0;
            px.seen[1] = 0;
            v2f raw[KB][8];
            auto fetch = [&](int kb) __attribute__((always_inline)) {
#pragma unroll
                for (int i = 0; i < 8; ++i) raw[kb][i] = buf_load2(ri, vi, (uint32_t)(kb * 16 + i) * row_bytes);
            };
            // two blocks in flight: with all of them the registers run out
            fetch(0);
            if (KB > 1) fetch(KB > 1 ? 1 : 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
                for (int nb = 0; nb < 2; ++nb) {
                    SplitUnit<8> s;
                    s.seen = px.seen[nb];
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = raw[kb][i][nb];
                    static_for<0, SplitUnit<8>::STEPS>([&](auto st) __attribute__((always_inline)) { s.template step<decltype(st)::value>(v); });
                    px.seen[nb] = s.seen;
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl) px.b[nb][kb][pl] = (u32x4){s.p[pl][0], s.p[pl][1], s.p[pl][2], s.p[pl][3]};
                }
                if (kb + 2 < KB) fetch(kb + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            have = tile;
        }
        cur.vo = vo;
        cur.k0 = (int)g * 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[q] = buf_load4(rb, (uint32_t)(g * 32 + 8 * q + 4 * half) * 4u);
    };
    // a unit that met values the split cannot hold: once more on the fp32 matrix cores, operands from memory
    auto check_unit = [&](PointUnit &cur, bool bad) {
        bad = bad || lossy_filter || split_lossy(px.seen[0]) || split_lossy(px.seen[1]);
        if (__ballot(bad) == 0) return;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) cur.acc[nb][r] = 0.f;
#pragma unroll 1
        for (int c = 0; c < C; c += 2) {
            const float a = buf_load1(rw, (uint32_t)((cur.k0 + j) * C + c + half) * 4u);
            const v2f b = buf_load2(ri, vi0 == kOobOffset ? kOobOffset : vi0 + (uint32_t)(c + half) * row_bytes, 0);
            cur.acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b.x, cur.acc[0], 0, 0, 0);
            cur.acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b.y, cur.acc[1], 0, 0, 0);
        }
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
            for (int r = 0; r < 16; ++r) cur.acc[nb][r] += bias[r >> 2][r & 3];
    };
    auto next_unit = [&]() {
        if (++g == (uint32_t)p.groups) { g = 0; ++tile; }
    };
    PointUnit A, B;
    uint32_t left = end - u;
    open_unit(A);
    check_unit(A, point_unit<KB, ACT, false>(At + half * K + g * 32 + j, K, px, bias, A, ro, row_bytes, A));
    next_unit();
    --left;
    while (left >= 2) {
        open_unit(B);
        check_unit(B, point_unit<KB, ACT, true>(At + half * K + g * 32 + j, K, px, bias, B, ro, row_bytes, A));
        next_unit();
        open_unit(A);
        check_unit(A, point_unit<KB, ACT, true>(At + half * K + g * 32 + j, K, px, bias, A, ro, row_bytes, B));
        next_unit();
        left -= 2;
    }
    if (left == 1) {
        open_unit(B);
        check_unit(B, point_unit<KB, ACT, true>(At + half * K + g * 32 + j, K, px, bias, B, ro, row_bytes, A));
        point_store<ACT>(ro, row_bytes, B, 0, 16);
    } else {
        point_store<ACT>(ro, row_bytes, A, 0, 16);
    }
}

// KB = C / 16.  512 threads, one workgroup per compute unit (its eight waves share one copy of the filter).
// LDS: At[kb][part][half][K] units, channels 16 kb + 8 half + 0..7 of an output channel.
constexpr int kPointThreads = 512;
template <int KB>
__global__ __launch_bounds__(kPointThreads, 2) void conv_point_kernel(const ConvPointKArgs p)
{
    extern __shared__ __attribute__((aligned(16))) u32x4 At[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // the same in all lanes: keeps unit bookkeeping scalar
    const int half = lane >> 5, j = lane & 31;
    const int K = p.K, C = KB * 16;

    bool lossy = false;
    {
        const __amdgpu_buffer_rsrc_t rw = make_rsrc(p.wt, (uint64_t)K * C * 4);
        for (int idx = tid; idx < K * KB * 2; idx += kPointThreads) {   // K is a multiple of 64: a wave has one octet
            const int o = idx / K, k = idx - o * K;
            const v4f v0 = buf_load4(rw, (uint32_t)(k * C + o * 8) * 4u), v1 = buf_load4(rw, (uint32_t)(k * C + o * 8 + 4) * 4u);
            const float v[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
            SplitUnit<8> s;
            static_for<0, SplitUnit<8>::STEPS>([&](auto st) __attribute__((always_inline)) { s.template step<decltype(st)::value>(v); });
            lossy |= split_lossy(s.seen);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                At[(((o >> 1) * 3 + pl) * 2 + (o & 1)) * K + k] = (u32x4){s.p[pl][0], s.p[pl][1], s.p[pl][2], s.p[pl][3]};
        }
    }
    lossy = __syncthreads_or(lossy);

    const uint32_t w = blockIdx.x * (kPointThreads / 64) + wave;
    const uint32_t u = w * p.per + (w < p.rem ? w : p.rem);
    const uint32_t end = u + p.per + (w < p.rem ? 1u : 0u);
    if (u >= end) return;
    if (p.act == POLYDL_ACT_NONE) point_run<KB, POLYDL_ACT_NONE>(p, At, lossy, u, end, half, j);
    else if (p.act == POLYDL_ACT_RELU) point_run<KB, POLYDL_ACT_RELU>(p, At, lossy, u, end, half, j);
    else point_run<KB, POLYDL_ACT_RELU6>(p, At, lossy, u, end, half, j);
}

bool conv_point_fits(const ConvProblem &q)
{
    const int64_t HW = (int64_t)q.H * q.W;
    if (q.R != 1 || q.S != 1 || q.stride != 1 || q.pad != 0 || q.pre_act != POLYDL_ACT_NONE) return false;
    if (q.C != 16 && q.C != 32 && q.C != 64) return false;
    // at least four channel groups share the pixels a wave holds (with 64 output channels the kernel
    // measured no faster than the staged one); the split filter has to fit 96 KB of LDS
    if (q.K % 64 != 0 || q.K < 128 || (int64_t)q.K * q.C > 16384) return false;
    if (HW % 2 != 0) return false;
    // every byte offset, tile base and unit count stays below 2^31
    if ((int64_t)q.N * HW * q.C * 4 >= 0x7FFFFFF0ll || (int64_t)q.N * HW * q.K * 4 >= 0x7FFFFFF0ll) return false;
    return true;
}

// waves of the grid and units per wave for this problem
void conv_point_shape(const ConvProblem &q, int cus, uint32_t *units, uint32_t *workgroups)
{
    const int64_t total = (int64_t)q.N * q.H * q.W;
    const uint32_t tiles = (uint32_t)((total + 63) / 64);
    *units = tiles * (uint32_t)(q.K / 32);
    const uint32_t fit = (uint32_t)cus;                      // one workgroup per compute unit (LDS)
    const uint32_t need = (*units + kPointThreads / 64 - 1) / (kPointThreads / 64);
    *workgroups = need < fit ? need : fit;
}

template <int KB>
static hipError_t launch_point(const ConvPointKArgs &a, uint32_t wgs, hipStream_t stream)
{
    const size_t lds = (size_t)a.K * KB * 16 * 6;
    if (lds > 64 * 1024) {   // more than the default window has to be asked for
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(conv_point_kernel<KB>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
        if (e != hipSuccess) return e;
    }
    return launch_kernel(conv_point_kernel<KB>, dim3(wgs), dim3(kPointThreads), lds, stream, a);
}

hipError_t conv_point_launch(const ConvProblem &q, hipStream_t stream)
{
    if (!conv_point_fits(q)) return hipErrorInvalidValue;
    ConvPointKArgs a;
    a.in = (const float *)q.in; a.wt = (const float *)q.wt; a.bias = q.bias; a.out = q.out;
    a.N = q.N; a.C = q.C; a.K = q.K; a.HW = q.H * q.W;
    a.groups = q.K / 32;
    uint32_t wgs;
    conv_point_shape(q, compute_units(), &a.units, &wgs);
    const uint32_t waves = wgs * (kPointThreads / 64);
    a.per = a.units / waves;
    a.rem = a.units % waves;
    a.recip_groups = div_recip((uint32_t)a.groups);
    a.recip_HW = div_recip((uint32_t)a.HW);
    a.act = q.act;
    if (q.C == 64) return launch_point<4>(a, wgs, stream);
    if (q.C == 32) return launch_point<2>(a, wgs, stream);
    return launch_point<1>(a, wgs, stream);
}

}  // namespace polydl
