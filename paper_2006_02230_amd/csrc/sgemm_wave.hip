// SGEMM of small products (wave_core.hpp).
#include "wave_core.hpp"

namespace polydl {

struct SgemmWaveKArgs {
    const float *A, *B;
    float *C;
    int M, N, K;
    WaveOrder order;
    WaveParts parts;
    float alpha, beta;         // C = beta*C + alpha*A*B; beta == 0 writes C without reading it
};

// B operand: row-major [K][N].
template <class T>
struct WaveBRows {
    static constexpr int PER_ROW = T::WN / 4, ROWS = 64 / PER_ROW, LOADS = 16 / ROWS;
    const char *base;
    uint32_t row_bytes, row_rest, off[LOADS];   // row_rest: bytes from the tile's first column to the end of a row
    int K;
    __amdgpu_buffer_rsrc_t rsrc;                // of the step being fetched
    __device__ __forceinline__ void init(const float *B, int n0, int N, int K_, int lane)
    {
        K = K_;
        base = reinterpret_cast<const char *>(B + n0);
        row_rest = (uint32_t)(N - n0) * 4u;
        row_bytes = (uint32_t)N * 4u;
        const int col = lane % PER_ROW * 4;
#pragma unroll
        for (int n = 0; n < LOADS; ++n) off[n] = n0 + col < N ? (uint32_t)(n * ROWS + lane / PER_ROW) * row_bytes + 4u * col : kOobOffset;
    }
    // rows past the end lie out of range
    __device__ __forceinline__ void begin(int t, bool live)
    {
        const uint32_t k = live ? 16u * (uint32_t)t : 0u, rows = min((uint32_t)K - k, 16u);
        rsrc = raw_rsrc(base + (uint64_t)k * row_bytes, live ? (rows - 1u) * row_bytes + row_rest : 0u);
    }
    template <int N>
    __device__ __forceinline__ void load(v4f *dst) const { lds_load<16>(rsrc, dst + N * 64, off[N]); }
    __device__ __forceinline__ void finish(float (&)[8]) const {}
};

template <class T>
__global__ __launch_bounds__(T::THREADS, T::WAVES_PER_SIMD) void sgemm_wave_kernel(SgemmWaveKArgs p)
{
    extern __shared__ __attribute__((aligned(16))) v4f slices[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tn;
    wave_tile(p.order, blockIdx.x, tm, tn);
    const int m0 = tm * T::WM, n0 = tn * T::WN;
    const int first = blockIdx.y * p.parts.part_steps, last = min(p.parts.steps, first + p.parts.part_steps);
    v16f acc[T::MB][T::NB];
    {
        WaveA<T> al;
        WaveBRows<T> bl;
        al.init(p.A, m0, p.M, p.K, lane);
        bl.init(p.B, n0, p.N, p.K, lane);
        wave_products<T>(al, bl, acc, first + wave, last, p.K, slices + wave * T::SLICE, lane);
    }
    wave_finish<T>(slices, acc, p.parts, wave, lane, [&](int u, const v4f (&v)[T::NB]) __attribute__((always_inline)) {
        const int col = n0 + (lane & 31), row = m0 + 32 * (u / 4) + 8 * (u % 4) + 4 * (lane >> 5);
        const uint64_t panel = (uint64_t)m0 * p.N * 4;
        const __amdgpu_buffer_rsrc_t rc = make_rsrc(reinterpret_cast<char *>(p.C) + panel, (uint64_t)p.M * p.N * 4 - panel);
        const uint32_t off = ((uint32_t)(row - m0) * (uint32_t)p.N + (uint32_t)col) * 4u, row_bytes = (uint32_t)p.N * 4u;
        uint32_t at[4][T::NB];      // out of range where the element is
        float c0[4][T::NB];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj) {
                at[e][bj] = row + e < p.M && col + 32 * bj < p.N ? off + 128u * bj : kOobOffset;
                c0[e][bj] = 0.f;
            }
        if (p.beta != 0.f) {   // uniform
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int bj = 0; bj < T::NB; ++bj) c0[e][bj] = buf_load1(rc, at[e][bj], e * row_bytes);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj) buf_store1(rc, at[e][bj], e * row_bytes, p.beta * c0[e][bj] + p.alpha * v[bj][e]);
    });
}

template <class T>
static hipError_t sgemm_wave_launch_t(const SgemmProblem &q, int parts, hipStream_t stream)
{
    SgemmWaveKArgs a;
    a.A = q.A; a.B = q.B; a.C = q.C;
    a.M = q.M; a.N = q.N; a.K = q.K;
    a.alpha = q.alpha; a.beta = q.beta;
    const int tiles_m = (q.M + T::WM - 1) / T::WM, tiles_n = (q.N + T::WN - 1) / T::WN, tiles = tiles_m * tiles_n;
    a.order = wave_order((uint32_t)tiles_m, (uint32_t)tiles_n);
    const hipError_t e = wave_parts((q.K + 15) / 16, parts, tiles, sizeof(float) * T::WM * T::WN, q.arena, stream, &a.parts);
    if (e != hipSuccess) return e;
    return wave_launch<T, sgemm_wave_kernel<T>>(tiles, a.parts.parts, stream, a);
}

hipError_t sgemm_wave_launch(const SgemmProblem &q, int tile, int waves, int parts, hipStream_t stream)
{
    if (waves == 4) return sgemm_wave_launch_t<WaveTile<2, 2, 4>>(q, parts, stream);
    return tile == 64 ? sgemm_wave_launch_t<WaveTile<2, 2, 8>>(q, parts, stream) : sgemm_wave_launch_t<WaveTile<1, 1, 8>>(q, parts, stream);
}

}  // namespace polydl
