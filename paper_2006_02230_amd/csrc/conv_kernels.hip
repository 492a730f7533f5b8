// Forward convolution as an implicit GEMM on the matrix cores, fp32 or bfloat16 with split operands.
//
// The paper's convolution nest (figure "The 2-D Convolution code") contains a GEMM in its three
// inner loops; here the whole nest is one GEMM  out[K][N*P*Q] = wt[K][C*R*S] * X[C*R*S][N*P*Q]
// where X is the im2col view of the input, never materialised: its elements are gathered from
// the NCHW tensor while the B stage is filled.  Rows (output channels) come from the KCRS filter
// tensor, which already is a row-major K x (C*R*S) matrix.  Output columns (n, p, q) are
// contiguous in NKPQ for a fixed channel, so the accumulator tile is stored without a transpose.
// The element-wise tail (bias, ReLU / ReLU6) runs on the accumulators before the store: the
// peeled last reduction iteration of algorithm "Perform operator fusion".
#include "conv_gather.hpp"
#include "variants.hpp"

namespace polydl {

template <class T, int AVEC, int MODE>
__global__ __launch_bounds__(T::NT) void conv_kernel(ConvKArgs p)
{
    __shared__ __attribute__((aligned(16))) float lds[T::LDS_FLOATS];
    const int tid = threadIdx.x, wave = tid >> 6;
    const ConvPart c = conv_part<T>(p);
    const int wm0 = (wave % T::WAVES_M) * T::WM, wn0 = (wave / T::WAVES_M) * T::WN;

    // AVEC = 1 stands for filter rows that are not a multiple of four floats long or not 16-byte
    // aligned: vector loads all the same, with the reduction's tail masked.  AVEC = 2 (GATHER_POINT): rows as
    // for 4, but not whole stages long, so that the gather has to mind the tail
    ALoader<T, 4, AVEC == 1> al;
    BLoaderIm2col<T, MODE, false, AVEC != 4> bl;
    __shared__ uint2 ktab[MODE == GATHER_TABLE ? kTableRows : 1];
    bl.fill_table(p, tid, ktab, c.kbegin, c.kend);
    al.init(p.wt, tid, c.m0, p.K, p.Kg, p.Kg);
    bl.init(p, tid, c.n0);
    if constexpr (MODE == GATHER_TABLE) __syncthreads();

    v16f acc[T::MB][T::NB];
#pragma unroll
    for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
        for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;

    gemm_mainloop<T, false>(lds, al, bl, acc, c.kbegin, c.kend, tid, wm0, wn0);
    conv_finish<T, 1>(p, c, acc, tid, wm0, wn0);
}

// The same with the products formed on the bfloat16 matrix cores (split_core.hpp), for reductions of
// kSplitMinReduction and more.  Bound: the gathering and splitting of every input value once per tap, beside
// matrix instructions that leave two to three times less time for it than the fp32 ones did; hence larger
// tiles with fewer reduction parts win (128x128 split 2 where 64x64 with cut leftovers did).  Batch 32, us:
// 128 -> 128 3x3 with the filter copy 66 -> 54, 512 -> 512 3x3 79 -> 64, 1024 -> 2048 1x1/2 64 -> 53,
// 512 -> 512 3x3 at 28x28 910 -> 620 .. 690.  Launched back to back the small ones run at 2.1 .. 2.3 GHz with the matrix
// cores busy a third of the cycles, the last one at 1.95 GHz (power) with 0.56; without load on the card it is 2.4 GHz.
// KTAIL: see BLoaderIm2col.
template <class T, int MODE, bool KTAIL>
__global__ __launch_bounds__(T::NT, T::SPLIT_WAVES) void conv_split_kernel(ConvKArgs p)
{
    __shared__ __attribute__((aligned(16))) u32x4 lds[SplitTile<T>::LDS_BYTES / 16];
    typedef BLoaderIm2col<T, MODE, true, KTAIL> Gather;
    __shared__ __attribute__((aligned(16))) uint2 ktab[Gather::TABLE_ROWS];
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const ConvPart c = conv_part<T>(p);
    const int wm0 = (wave % T::WAVES_M) * T::WM, wn0 = (wave / T::WAVES_M) * T::WN;
    v16f acc[T::MB][T::NB];
    bool redo;
    {
        SplitALoader<T> al;
        Gather bl;
        bl.fill_table(p, tid, ktab, c.kbegin, c.kend);
        al.init(p.wt, tid, c.m0, p.K, p.Kg, p.Kg);
        bl.init(p, tid, c.n0);
        if constexpr (Gather::PERIODIC) __syncthreads();
        SplitAcc<T> sum;
        sum.clear();
        split_mainloop<T>(lds, al, bl, sum, c.kbegin, c.kend, tid, wm0, wave / T::WAVES_M);
        redo = sum.finish(acc) || al.lossy() || bl.lossy();
    }
    if (__syncthreads_or(redo)) {   // values the split cannot hold: once more on the fp32 matrix cores
        ALoader<T, 4, true> al;
        BLoaderIm2col<T, MODE> bl;
        al.init(p.wt, tid, c.m0, p.K, p.Kg, p.Kg);
        bl.init(p, tid, c.n0);
#pragma unroll
        for (int bi = 0; bi < T::MB; ++bi)
#pragma unroll
            for (int bj = 0; bj < T::NB; ++bj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[bi][bj][r] = 0.f;
        gemm_mainloop<T, false>(reinterpret_cast<float *>(lds), al, bl, acc, c.kbegin, c.kend, tid, wm0, wn0);
    }
    conv_finish<T, kPartsAhead<T>>(p, c, acc, tid, wm0, wn0);
}

template <class T>
static hipError_t conv_launch(const ConvProblem &q, int split_k, int raster, hipStream_t stream)
{
    static_assert(T::BK != 16 || (kSplitMinReduction / T::BK + 3) * T::BK <= kTableRows, "short reductions fit the table");
    ConvKArgs a;
    a.in = static_cast<const float *>(q.in); a.wt = static_cast<const float *>(q.wt);
    a.bias = q.bias; a.out = q.out;
    a.C = q.C; a.H = q.H; a.W = q.W; a.K = q.K; a.R = q.R; a.S = q.S;
    a.stride = q.stride; a.pad = q.pad; a.P = q.P; a.Q = q.Q;
    a.PQ = q.P * q.Q; a.RS = q.R * q.S; a.HW = q.H * q.W; a.CHW = q.C * q.H * q.W;
    a.Kg = q.C * q.R * q.S;
    a.Ng = q.N * a.PQ;
    a.magic_C = div_magic((uint32_t)q.C);
    a.magic_RS = div_magic((uint32_t)a.RS);
    a.magic_S = div_magic((uint32_t)q.S);
    a.one_RS = a.RS == 1 ? 0xFFFFFFFFu : 0u;
    a.one_S = q.S == 1 ? 0xFFFFFFFFu : 0u;
    a.in_bytes = (uint64_t)q.N * a.CHW * 4;
    a.out_bytes = (uint64_t)q.N * q.K * a.PQ * 4;
    a.recip_PQ = div_recip((uint32_t)a.PQ);
    a.recip_Q = div_recip((uint32_t)q.Q);
    a.tiles_m = (q.K + T::BM - 1) / T::BM;
    a.tiles_n = (a.Ng + T::BN - 1) / T::BN;
    int stages = (a.Kg + T::BK - 1) / T::BK;
    if (split_k < 1) split_k = 1;
    if (split_k > stages) split_k = stages;
    int stages_per = (stages + split_k - 1) / split_k;
    a.k_per_split = stages_per * T::BK;
    a.split_k = (stages + stages_per - 1) / stages_per;
    const bool tail = raster >= 2;   // rasters 2 and 3: tile order of raster 0 and 1, leftover tiles split
    a.raster = raster & 1;
    a.act = q.act;
    a.pre_act = q.pre_act;
    a.partials = nullptr;
    a.counters = nullptr;
    const int tiles = a.tiles_m * a.tiles_n;
    a.whole_tiles = tiles; a.tail_parts = 1; a.tail_k = a.k_per_split; a.recip_tail = 0;
    dim3 grid((unsigned)tiles, (unsigned)a.split_k), block(T::NT);
    size_t scratch = 0;   // partial tiles
    int cut_tiles = 0;
    if (a.split_k > 1) {
        scratch = (size_t)tiles * a.split_k * T::BM * T::BN * sizeof(float);
        cut_tiles = tiles;
    } else {
        // rasters 2, 3: an unsplit grid whose last round would leave most compute units idle has the
        // tiles of that round split
        const TailSplit ts = tail ? tail_split(tiles, stages, compute_units()) : TailSplit{0, 1, stages};
        if (ts.parts > 1) {
            a.whole_tiles = tiles - ts.tiles; a.tail_parts = ts.parts; a.tail_k = ts.stages_per_part * T::BK;
            a.recip_tail = div_recip((uint32_t)ts.parts);
            scratch = (size_t)ts.tiles * ts.parts * T::BM * T::BN * sizeof(float);
            cut_tiles = ts.tiles;
            grid = dim3((unsigned)(a.whole_tiles + ts.tiles * ts.parts), 1u);
        }
    }
    if (scratch > 0) {
        hipError_t e = splitk_scratch(stream, q.arena, scratch, cut_tiles, &a.partials, &a.counters);
        if (e != hipSuccess) return e;
    }
    const bool avec = (a.Kg % 4 == 0) && ((uintptr_t)q.wt % 16 == 0);
    // tile layout 2: the filter comes as [K][R][S][C], 16-byte aligned (its rows load as vectors)
    const bool tapmajor = q.wt_tap != nullptr;
    if (tapmajor) {
        if (!gather_tap_major_fits(q, T::BK) || ((uintptr_t)q.wt_tap & 15)) return hipErrorInvalidValue;
        a.wt = q.wt_tap;
    }
    const bool table = gather_table_fits(q, T::BK);
    const int mode = (q.R == 1 && q.S == 1 && q.pad == 0) ? GATHER_POINT
                     : tapmajor ? GATHER_TAPMAJOR
                     : table ? GATHER_TABLE
                     : a.RS <= 31 ? GATHER_TAPS1 : a.RS <= 63 ? GATHER_TAPS2 : GATHER_ANY;
    if constexpr (T::SPLIT) {
        if (split_pays(q.K, a.RS, a.Kg)) {
#define POLYDL_GO(MODE, KTAIL) return launch_kernel((conv_split_kernel<T, MODE, KTAIL>), grid, block, 0, stream, a)
            switch (mode) {
            case GATHER_TAPMAJOR: POLYDL_GO(GATHER_TAPMAJOR, true);
            case GATHER_POINT:
                if (a.Kg % T::BK == 0) POLYDL_GO(GATHER_POINT, false);
                POLYDL_GO(GATHER_POINT, true);
            default:
                if (a.RS <= 31) POLYDL_GO(GATHER_TAPS1, true);
                if (a.RS <= 63) POLYDL_GO(GATHER_TAPS2, true);
                POLYDL_GO(GATHER_ANY, true);
            }
#undef POLYDL_GO
        }
    }
#define POLYDL_GO(AV, MODE) return launch_kernel((conv_kernel<T, AV, MODE>), grid, block, 0, stream, a)
    if (mode == GATHER_TAPMAJOR) POLYDL_GO(4, GATHER_TAPMAJOR);
    if (avec) {
        if (mode == GATHER_POINT && a.Kg % T::BK == 0) POLYDL_GO(4, GATHER_POINT);
        if (mode == GATHER_POINT) POLYDL_GO(2, GATHER_POINT);
        if (mode == GATHER_TABLE) POLYDL_GO(4, GATHER_TABLE);
    } else {
        if (mode == GATHER_POINT) POLYDL_GO(1, GATHER_POINT);
        if (mode == GATHER_TABLE) POLYDL_GO(1, GATHER_TABLE);
    }
    if constexpr (!T::SPLIT) {   // reductions the other tiles come here with fit the table (or take GATHER_ANY)
        if (avec) {
            if (mode == GATHER_TAPS1) POLYDL_GO(4, GATHER_TAPS1);
            if (mode == GATHER_TAPS2) POLYDL_GO(4, GATHER_TAPS2);
        } else {
            if (mode == GATHER_TAPS1) POLYDL_GO(1, GATHER_TAPS1);
            if (mode == GATHER_TAPS2) POLYDL_GO(1, GATHER_TAPS2);
        }
    }
    if (avec) POLYDL_GO(4, GATHER_ANY);
    POLYDL_GO(1, GATHER_ANY);
#undef POLYDL_GO
}

#define POLYDL_DEFINE_CONV(BM, BN, BK, WM, WN)                                                            \
    hipError_t conv_launch_##BM##x##BN##x##BK##_##WM##x##WN(const ConvProblem &q, int s, int r,           \
                                                            hipStream_t st)                              \
    {                                                                                                    \
        return conv_launch<Tile<BM, BN, BK, WM, WN>>(q, s, r, st);                                        \
    }
POLYDL_TILE_FAMILY(POLYDL_DEFINE_CONV)

}  // namespace polydl
