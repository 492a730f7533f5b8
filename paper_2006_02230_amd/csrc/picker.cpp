// Tile-configuration picker: the paper's reuse analysis re-derived for the CDNA4 memory hierarchy.
//
// PolyDL ranks loop-nest variants without running them (section "Compile Time Selection of Top
// performing code version"): algorithm "Compute working set sizes" lists, per data reuse, how much
// data is touched between the source and the target of the reuse; algorithm "Compute working set
// sizes w.r.t cache sizes" places every working set in the fastest level it fits; equation (1)
// charges each level's working sets with that level's cost per byte.  Here the variants are the
// compiled tile family, the loop nest is fixed (workgroup tile around a register-resident wave
// tile), so the working sets have closed forms, and the levels are accumulator registers, LDS,
// the XCD's L2 and the Infinity Cache, with HBM as memory.
//
// Two additions the GPU needs, both stated by the paper as requirements of a good schedule
// (section "Introduction": load-balanced parallel loops; section "The GEMM microkernel": the
// microkernel must keep the vector/matrix unit busy):
//   * a matrix-core term: the MFMA cycles of the busiest SIMD after the workgroups are dealt to
//     256 compute units, divided by an issue efficiency that depends on the wave tile and the
//     stage depth;
//   * the data term weights each reuse by the bytes that actually travel (the operand panel times
//     the number of times it is fetched) instead of by the working-set size alone.
// The predicted time is max(matrix-core term, data term) + fixed costs; the lowest wins, as in
// the paper's ranking (lower cost = higher rank).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>
#include "internal.hpp"

namespace polydl {

// ---- hardware table (MI355X; capacities are public figures, rates are measured or assumed) -----
struct Level {
    const char *name;
    double capacity;      // bytes available to one reuse scope at this level
    double gbytes_per_s;  // aggregate rate the whole chip sustains from this level
};
static Level kLevels[4] = {
    {"acc", 64.0 * 1024, 1e9},              // accumulator registers of one wave (256 regs x 64 lanes)
    {"lds", 80.0 * 1024, 60000.0},          // half of a CU's 160 KB: two workgroups share a CU
    {"l2", 4.0 * 1024 * 1024, 16000.0},     // one XCD's L2
    {"mall", 256.0 * 1024 * 1024, 8000.0},  // Infinity Cache
};
static double kHbmGBs = 4500.0;             // sustained mixed read/write HBM rate

void model_get_levels(double *capacity, double *gbytes_per_s, double *mem_gbytes_per_s)
{
    for (int i = 0; i < 4; ++i) { capacity[i] = kLevels[i].capacity; gbytes_per_s[i] = kLevels[i].gbytes_per_s; }
    *mem_gbytes_per_s = kHbmGBs;
}
void model_set_levels(const double *capacity, const double *gbytes_per_s, double mem_gbytes_per_s)
{
    for (int i = 0; i < 4; ++i) { kLevels[i].capacity = capacity[i]; kLevels[i].gbytes_per_s = gbytes_per_s[i]; }
    kHbmGBs = mem_gbytes_per_s;
}
static const double kClockHz = 2.4e9;
// Gather cost per element with the filter copy of tile layout 2, relative to layout 0 (fitted to a
// sweep of the 3x3 layers of the ResNet-50-shaped suite).
static const double kTapMajorGather = 0.5, kTapMajorGather11 = 0.3, kTapMajorGather21 = 0.6;
static const int kSimdsPerCU = 4, kXcds = 8;
// compute units of the current device (256 on an MI355X; also the answer when no device is visible)
#define kCUs (compute_units())

// Algorithm "Compute working set sizes w.r.t cache sizes".  placed (may be null) receives, per
// working set in the caller's order, the level it went to (nlevels = memory).
static void bucket_placed(int n, const double *ws, int nlevels, const double *sizes, double *levels, double *mem,
                          int *placed)
{
    std::vector<int> order(n);
    for (int i = 0; i < n; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return ws[a] < ws[b]; });
    for (int i = 0; i < nlevels; ++i) levels[i] = 0;
    *mem = 0;
    for (int idx : order) {
        int at = nlevels;
        for (int i = 0; i < nlevels && at == nlevels; ++i)
            if (ws[idx] + levels[i] <= sizes[i]) at = i;
        if (at < nlevels) levels[at] += ws[idx];
        else *mem += ws[idx];
        if (placed) placed[idx] = at;
    }
}

void reuse_bucket(int n, const double *ws, int nlevels, const double *sizes, double *levels, double *mem)
{
    bucket_placed(n, ws, nlevels, sizes, levels, mem, nullptr);
}

double reuse_cost(int nlevels, const double *levels, double mem, const double *weights, double mem_weight)
{
    double c = mem * mem_weight;
    for (int i = 0; i < nlevels; ++i) c += levels[i] * weights[i];
    return c;
}

static double rate_of(int level) { return level < 4 ? kLevels[level].gbytes_per_s : kHbmGBs; }

struct Shape {   // the GEMM a candidate works on
    double Mg, Ng, Kg;           // output rows, output columns, reduction length (padded as executed)
    double a_bytes, b_bytes, d_bytes;   // operand and result tensors
    double b_tile_bytes;         // B-side bytes one workgroup fetches for its whole reduction
};

struct Cand {
    int bm, bn, wm, wn, threads;
    int split_k;
    double steps_per_stage;      // MFMA k-steps between two barriers
    double lds_bytes;
    double loop_eff;             // matrix-core share of the reduction loop's time, large wave tile, deep stage
    double wg_overhead_cycles;   // cycles a wave spends outside the reduction loop (setup, first loads, stores)
    double kernel_fixed_us;      // launch, first-stage latency and the store tail that nothing overlaps
    int max_waves_per_simd;
    // Convolution kernels are timed round by round (see model()): workgroups that are resident
    // together start, load and store in step, so each round pays its own latency.
    bool rounds = false;
    int regs = 128;              // vector registers the compiler reports for the instantiation
    double eff_sat = 0.65;       // matrix-core share of a stage once enough workgroups share a SIMD
    double t_lat_us = 0.8;       // a stage is never shorter than one global-to-LDS round trip
    double t_round_us = 8.0;     // per round: setup, first loads, epilogue of the last workgroup
    double gather_elems = 0;     // B elements a thread gathers per stage (im2col addressing in the ALUs)
    double gather_cycles = 0;    // cycles of that addressing per element
    double split_c0 = 0, split_c1 = 0;   // split reduction: microseconds, and microseconds per MB of parts
    // Tiles whose products run on the bfloat16 matrix cores (split_core.hpp): six 32-cycle instructions per 16
    // reduction steps instead of eight of 64; split_eff is the matrix-core share of their loop.
    bool split = false;
    double split_eff = 0.4;
    double split_overhead = 0;   // cycles of a workgroup's prologue and epilogue (SGEMM)
    double read_overhead = 0;    // and of an epilogue that reads C first
    double tail_us = 4.0;        // leftover tiles cut into parts: the hand-over
    double sum_us = 0;           // split reduction: the last part of a tile adds all parts alone
    bool tail_split = false;     // the kernel cuts the leftover tiles of an unsplit grid (tail_split())
};

// Constants below were fitted to an exhaustive sweep of the compiled family on the ResNet-50-shaped
// suite (time against reduction length, workgroup count and wave tile).
static void model(const Shape &s, const Cand &c, polydl_model_report *r)
{
    std::memset(r, 0, sizeof(*r));
    const double tiles_m = std::ceil(s.Mg / c.bm), tiles_n = std::ceil(s.Ng / c.bn);
    const double wgs = tiles_m * tiles_n * c.split_k;
    const double waves_per_wg = c.threads / 64.0;
    const double mb = c.wm / 32.0, nb = c.wn / 32.0;
    // ---- matrix-core term -----------------------------------------------------------------
    // Workgroups are dealt to the 256 CUs; a SIMD runs the waves it is given one after another
    // (two at a time share its matrix core), so the busiest SIMD sets the time: this is the
    // load-balance requirement on the parallel loops.
    const double steps = std::ceil(s.Kg / 2.0 / c.split_k);               // rank-2 updates per wave
    const double step_cycles = c.split ? 24.0 : 64.0;                     // matrix-core cycles of one, per block
    const double wgs_on_busiest_cu = std::ceil(wgs / kCUs);
    const double waves_on_busiest_simd = std::ceil(wgs_on_busiest_cu * waves_per_wg / kSimdsPerCU);
    double resident = std::min<double>(c.max_waves_per_simd, std::floor(2.0 * kLevels[1].capacity / c.lds_bytes) *
                                                                 waves_per_wg / kSimdsPerCU);
    resident = std::max(1.0, std::min(resident, waves_on_busiest_simd));
    // issue efficiency: small wave tiles spend more issue slots per MFMA on operand reads and
    // address updates; every stage pays a barrier and an LDS round trip; a SIMD holding a single
    // wave cannot hide either
    double eff = c.loop_eff * (1.0 - 0.16 / (mb * nb));
    eff *= c.steps_per_stage / (c.steps_per_stage + 1.0 / (mb * nb));
    if (resident < 2) eff *= 0.72;
    else if (resident * mb * nb < 4) eff *= 0.85;   // two small waves leave gaps a third would fill
    if (c.split) eff = c.split_eff * (resident < 2 ? 0.666 : 1.0);
    // setup plus an epilogue that grows with the accumulators a lane has to store
    const double overhead = c.split ? c.split_overhead : c.wg_overhead_cycles * (0.3 + 0.7 * mb * nb / 2.0);
    const double wave_cycles = steps * mb * nb * step_cycles / eff + overhead + c.read_overhead;
    double mfma_us = waves_on_busiest_simd * wave_cycles / kClockHz * 1e6;
    if (c.rounds) {
        // Resident workgroups per CU, from registers (512 per SIMD lane, at most 8 waves per SIMD)
        // and LDS (160 KB).  The grid runs in rounds of that many workgroups per CU; within a
        // round the workgroups of a CU share its matrix cores stage by stage, and a round ends
        // with the epilogue of its workgroups before the next one's first loads are issued.
        const int waves_per_simd = std::min(8, 512 / ((c.regs + 7) / 8 * 8));
        const double by_regs = std::floor(waves_per_simd * kSimdsPerCU / waves_per_wg);
        const double by_lds = std::floor(160.0 * 1024 / c.lds_bytes);
        const double occ = std::max(1.0, std::min(by_regs, by_lds));
        double per_cu = wgs / kCUs;
        const double stages_all = std::ceil(steps / c.steps_per_stage);
        // leftover tiles cut into pieces: whole tiles are dealt evenly, the pieces make a short tail
        double tail_us = 0;
        if (c.tail_split && c.split_k == 1 && wgs < 2e9) {
            const TailSplit ts = tail_split((int)wgs, (int)stages_all, kCUs);
            if (ts.parts > 1) {
                per_cu = (wgs - ts.tiles) / kCUs;
                const double pieces = std::ceil((double)ts.tiles * ts.parts / kCUs);
                const double simd_share0 = std::ceil(waves_per_wg / kSimdsPerCU);
                tail_us = c.tail_us + pieces * ts.stages_per_part *
                                    (c.steps_per_stage * mb * nb * step_cycles * simd_share0 / kClockHz * 1e6 / c.eff_sat +
                                     c.gather_elems * c.gather_cycles / kClockHz * 1e6);
            }
        }
        const double full_rounds = std::floor(per_cu / occ);
        const double rest = per_cu - full_rounds * occ;
        const double stages = std::ceil(steps / c.steps_per_stage);
        const double simd_share = std::ceil(waves_per_wg / kSimdsPerCU);
        const double t_stage = c.steps_per_stage * mb * nb * step_cycles * simd_share / kClockHz * 1e6 / c.eff_sat +
                               c.gather_elems * c.gather_cycles / kClockHz * 1e6;
        auto round_us = [&](double n) { return c.t_round_us + stages * std::max(n * t_stage, c.t_lat_us); };
        mfma_us = full_rounds * round_us(occ) + (rest > 1e-9 ? round_us(std::ceil(rest - 1e-9)) : 0.0) + tail_us;
    }
    // ---- the reuses of the nest: working set (bytes) and the bytes that travel because of it ----
    // Algorithm 2 places the working sets, smallest first, each in the fastest level that still
    // has room beside those already there; a reuse whose working set was placed in level L is
    // served from L, so its traffic is charged at L's rate: equation (1) with each level's term
    // weighted by the bytes that actually move instead of by the working-set size alone.
    enum { R_ACC = 0, R_STAGE, R_COL_STEP, R_PAR, R_ALL, N_REUSE };
    const double a_panel = c.bm * s.Kg * 4;                                // A row panel between two column tiles
    // reuse across workgroups that run together on one XCD (the dependence spans the parallel
    // loop): the footprint of everything resident there
    const double res_wgs = std::min(wgs, (double)kCUs / kXcds * std::max(1.0, resident * kSimdsPerCU / waves_per_wg));
    const double dm = std::min(tiles_m, res_wgs), dn = std::max(1.0, std::ceil(res_wgs / tiles_m));
    double ws[N_REUSE], traffic[N_REUSE];
    ws[R_ACC] = (double)c.wm * c.wn * 4;                                   // accumulators over the reduction
    ws[R_STAGE] = c.lds_bytes;                                             // staged operands, shared by the waves
    ws[R_COL_STEP] = a_panel + s.b_tile_bytes + (double)c.bm * c.bn * 4;   // one column-tile step: A panel reused by the next
    ws[R_PAR] = dm * a_panel + dn * s.b_tile_bytes;                        // B tile (and A panels) shared by concurrent tiles
    ws[R_ALL] = s.a_bytes + s.b_bytes + s.d_bytes;                         // the tensors themselves
    // A is fetched once per column tile, B once per row tile; the accumulators never leave the
    // registers; every staged element is read from LDS once per wave that multiplies it
    const double a_traffic = tiles_n * s.a_bytes, b_traffic = tiles_m * tiles_n * s.b_tile_bytes;
    traffic[R_ACC] = 0;
    traffic[R_STAGE] = tiles_m * tiles_n * s.Kg * ((double)c.bm * (c.bn / c.wn) + (double)c.bn * (c.bm / c.wm)) * 4;
    traffic[R_COL_STEP] = a_traffic - s.a_bytes;
    traffic[R_PAR] = b_traffic > s.b_bytes ? b_traffic - s.b_bytes : 0;
    traffic[R_ALL] = s.a_bytes + s.b_bytes + s.d_bytes;
    double sizes[4], weights[4];
    for (int i = 0; i < 4; ++i) { sizes[i] = kLevels[i].capacity; weights[i] = 1.0 / kLevels[i].gbytes_per_s; }
    int placed[N_REUSE];
    bucket_placed(N_REUSE, ws, 4, sizes, r->level_bytes, &r->mem_bytes, placed);
    r->eq1_cost = reuse_cost(4, r->level_bytes, r->mem_bytes, weights, 1.0 / kHbmGBs);
    r->n_ws = N_REUSE;
    for (int i = 0; i < N_REUSE; ++i) { r->ws[i] = ws[i]; r->ws_level[i] = placed[i]; r->ws_traffic[i] = traffic[i]; }
    // ---- data term ------------------------------------------------------------------------------
    // Nothing faster than L2 is shared between workgroups, and nothing faster than the Infinity
    // Cache holds a tensor from one launch to the next: reuses across workgroups are served from
    // their placed level or L2, whichever is slower; the tensors from theirs or the Infinity Cache.
    const int a_level = std::max(2, placed[R_COL_STEP]), b_level = std::max(2, placed[R_PAR]);
    const int all_level = std::max(3, placed[R_ALL]);
    const double refetch_us = traffic[R_COL_STEP] / rate_of(a_level) * 1e-3 + traffic[R_PAR] / rate_of(b_level) * 1e-3;
    const double lds_us = traffic[R_STAGE] / rate_of(std::max(1, placed[R_STAGE])) * 1e-3;
    double mem_us = traffic[R_ALL] / rate_of(all_level) * 1e-3;            // compulsory
    if (c.rounds) mem_us = std::max(mem_us, refetch_us);                   // caches and memory work side by side
    else mem_us += refetch_us;
    mem_us = std::max(mem_us, lds_us);
    double fixed = c.kernel_fixed_us;
    if (c.rounds) {
        // nothing streams the tensors faster than this, with the first and last touches exposed
        mem_us = std::max(mem_us, (s.a_bytes + s.b_bytes + s.d_bytes) / 5500.0 * 1e-3 + 2.0);
        // a layer that mostly writes is slower than that: measured on the pointwise layers of the
        // suite (batch 16 .. 128, either kernel), the output leaves at about 3.15 TB/s
        mem_us = std::max(mem_us, (s.a_bytes + s.b_bytes) / 20000.0 * 1e-3 + s.d_bytes / 3150.0 * 1e-3 + 2.0);
        if (c.split_k > 1) fixed += c.split_c0 + c.split_c1 * c.split_k * s.d_bytes * 1e-6 + c.sum_us;
    } else if (c.split_k > 1) {
        // every part writes its accumulator tile once, coalesced; the last part of each tile reads
        // them all back and runs the epilogue: no other launch, no pass over the output
        fixed += 2.0 * c.split_k * s.d_bytes / kHbmGBs * 1e-3;
    }
    r->mfma_us = mfma_us;
    r->mem_us = mem_us;
    r->fixed_us = fixed;
    r->predicted_us = std::max(mfma_us, mem_us) + fixed;
    r->workgroups = (int)std::min(wgs, 2e9);
    r->simd_load = waves_on_busiest_simd;
}

// ---- convolution ---------------------------------------------------------------------------------
// filters of five rows or more are staged one filter row at a time by the patch kernel
static int patch_rows_per_stage(const ConvProblem &q) { return q.R >= 5 ? 1 : q.R; }

static double conv_patch_rows(const ConvProblem &q, int bn)
{
    const double Rp = patch_rows_per_stage(q);
    const double PQ = (double)q.P * q.Q, Ng = q.N * PQ;
    const double run = std::min<double>(bn, Ng);
    const double rows_out = std::min<double>(std::ceil((run - 1) / q.Q) + 1, (double)q.N * q.P);
    const double imgs = std::min<double>(std::ceil((run - 1) / PQ) + 1, q.N);
    const double prs = Rp == 1 ? 1 : q.stride;
    return rows_out * prs + imgs * std::max(0.0, Rp - prs);
}

static Shape conv_shape(const ConvProblem &q, int algo, int bn, int cb)
{
    Shape s;
    const double RS = (double)q.R * q.S;
    s.Mg = q.K;
    s.Ng = (double)q.N * q.P * q.Q;
    const double cexec = algo == 1 ? std::ceil((double)q.C / cb) * cb : q.C;
    s.Kg = cexec * RS;
    s.a_bytes = (double)q.K * q.C * RS * 4;
    s.b_bytes = (double)q.N * q.C * q.H * q.W * 4;
    s.d_bytes = (double)q.N * q.K * q.P * q.Q * 4;
    if (algo == 1) {
        const double wp = q.S == 1 ? q.Q : q.W + 2 * q.pad;
        // rows staged once per channel (once per channel and filter row when staged row by row)
        s.b_tile_bytes = q.C * conv_patch_rows(q, bn) * wp * 4 * (q.R / patch_rows_per_stage(q));
    } else {
        s.b_tile_bytes = (double)bn * q.C * RS * 4;                        // every tap gathered again
    }
    return s;
}

void model_conv(const ConvProblem &q, const polydl_tile_cfg &cfg, int threads, int reg_class, polydl_model_report *r)
{
    Cand c;
    c.bm = cfg.bm; c.bn = cfg.bn; c.wm = cfg.wm; c.wn = cfg.wn; c.threads = threads;
    c.split_k = std::max(1, cfg.split_k);
    if (cfg.algo == 1) {
        const int cb = std::max(2, cfg.cb);
        const double wp = q.S == 1 ? q.Q : q.W + 2 * q.pad;
        const double RSp = (double)patch_rows_per_stage(q) * q.S;     // taps of a channel in one stage
        c.steps_per_stage = cb / 2.0 * RSp;
        // two stage buffers, one when a workgroup's share of the reduction is a single stage
        const int nstages = (q.C + cb - 1) / cb * (q.R / patch_rows_per_stage(q));
        const int per_split = (nstages + c.split_k - 1) / c.split_k;
        c.lds_bytes = (per_split > 1 ? 2.0 : 1.0) * (cfg.bm * (cb * RSp + 1) + cb * conv_patch_rows(q, cfg.bn) * wp) * 4;
        c.loop_eff = 0.74;
        c.wg_overhead_cycles = 9000;
        c.kernel_fixed_us = 14.0;
        // the small-register instantiation holds 5 waves per SIMD with a 32x32 wave tile, 3 with
        // 64x32 in the 128x64 tile; everything else 2
        c.max_waves_per_simd = 2;
        if (reg_class >= 1 && cfg.wm * cfg.wn == 32 * 32) {
            c.max_waves_per_simd = 5;      // enough waves to cover each other's loads and stores
            c.loop_eff = 0.92;
            c.wg_overhead_cycles = 4000;
        }
        else if (reg_class >= 1 && cfg.bm == 128 && cfg.bn == 64) c.max_waves_per_simd = 3;
        // fitted on the sweep, by wave tile
        const int mbn = (cfg.wm / 32) * 10 + cfg.wn / 32;
        const int rc = reg_class < 0 ? 0 : reg_class;
        c.rounds = true;
        c.kernel_fixed_us = 5.0;
        if (mbn == 11)      { static const int R[3] = {192, 80, 60};   c.regs = R[rc]; c.eff_sat = 0.65; c.t_lat_us = 0.8; c.t_round_us = 6; }
        else if (mbn == 21) { static const int R[3] = {215, 110, 89};  c.regs = R[rc]; c.eff_sat = 0.60; c.t_lat_us = 0.6; c.t_round_us = 6; }
        else                { static const int R[3] = {247, 156, 121}; c.regs = R[rc]; c.eff_sat = 0.75; c.t_lat_us = 0.6; c.t_round_us = 6; c.split_c0 = 4; }
        c.split_c1 = 0.1;
    } else {
        c.steps_per_stage = cfg.bk / 2.0;
        c.lds_bytes = 2.0 * (cfg.bm * (cfg.bk + 4) + cfg.bk * (cfg.bn + 4)) * 4;
        c.loop_eff = 0.84;
        c.wg_overhead_cycles = 5000;
        c.kernel_fixed_us = 10.0;
        c.max_waves_per_simd = (cfg.wm * cfg.wn > 64 * 64) ? 1 : ((cfg.wm * cfg.wn == 64 * 64) ? 2 : 4);
        const int mbn = (cfg.wm / 32) * 10 + cfg.wn / 32;
        const bool point = q.R == 1 && q.S == 1 && q.pad == 0;   // loads without per-lane arithmetic
        c.rounds = true;
        c.kernel_fixed_us = 5.0;
        c.gather_elems = (double)cfg.bk * cfg.bn / threads;
        switch (mbn) {
        case 11: c.regs = 62;  c.eff_sat = 0.85; c.t_lat_us = 0.6; c.t_round_us = 2; c.gather_cycles = 32; c.split_c0 = 1; break;
        case 12: c.regs = 90;  c.eff_sat = 0.80; c.t_lat_us = 1.0; c.t_round_us = 4; c.gather_cycles = 20; c.split_c0 = 2; break;
        case 21: c.regs = 88;  c.eff_sat = 0.90; c.t_lat_us = 0.8; c.t_round_us = 4; c.gather_cycles = 40; c.split_c0 = 1; break;
        case 22: c.regs = cfg.bk == 16 ? 136 : 104; c.eff_sat = 0.80; c.t_lat_us = 0.8; c.t_round_us = 2; c.gather_cycles = 40;
                 c.split_c0 = 8; c.split_c1 = 0.2; break;
        case 24: c.regs = 212; c.eff_sat = 0.70; c.t_lat_us = 0.4; c.t_round_us = 2; c.gather_cycles = 20; c.split_c0 = 15; c.split_c1 = 0.6; break;
        default: c.regs = 228; c.eff_sat = 0.80; c.t_lat_us = 0.4; c.t_round_us = 4; c.gather_cycles = 20; c.split_c0 = 15; c.split_c1 = 1.0; break;
        }
        c.tail_split = cfg.raster >= 2;
        const bool split = split_products(cfg.bk, cfg.wm, cfg.wn) && split_pays(q.K, q.R * q.S, (int64_t)q.C * q.R * q.S);
        double point_gather = 0.1, tap_gather = mbn == 11 ? kTapMajorGather11 : (mbn == 21 ? kTapMajorGather21 : kTapMajorGather);
        double table_gather = 1, taps_gather = 1, taps_lat = 1;   // the split kernels': row table, and KCRS order
        if (split) {
            // fitted to sweeps of 97 problems (the suite at batch 1 .. 64 and the three held-out sets, with and without
            // the filter copy, reductions of 128 and more; small batches weighted): the picks run within 1.2 % of
            // the sweep's best on average, 8 % at worst.  The factors of short reductions (row table,
            // tiles of one and two blocks a wave) and of layers of at most 64 output channels in the KCRS order come
            // from 339 more layers of 16 .. 1024 channels on 7x7 .. 112x112 at batch 1 .. 64: the fit had too few of
            // those and left the reduction of 128 -> 64 3x3 on 56x56, batch 8, whole (56.5 us; in three parts 46.9).
            // For the others the same factors gained as much as they lost.
            c.split = true;
            c.lds_bytes = split_lds_bytes(cfg.bm, cfg.bn);
            point_gather = 0.29;
            if (mbn != 22) table_gather = 0.72;
            c.tail_us = 9.3;
            c.split_c1 = 0.078;
            c.sum_us = c.split_k * (double)cfg.bm * cfg.bn * 4 / (mbn == 11 ? 67.0 : 60.6) * 1e-3;
            switch (mbn == 22 && threads == 512 ? 0 : mbn) {
            case 11: c.regs = 128; taps_gather = 1.08; taps_lat = 0.99; c.eff_sat = 0.405; c.t_lat_us = 0.333; c.t_round_us = 2.07; c.gather_cycles = 43.4; tap_gather = 0.58; c.split_c0 = 0.85; c.tail_us = 4.8; break;
            case 12: c.regs = 168; taps_gather = 1.02; taps_lat = 1.34; c.eff_sat = 0.476; c.t_lat_us = 0.541; c.t_round_us = 2.07; c.gather_cycles = 46.9; tap_gather = 0.325; c.split_c0 = 2.17; break;
            case 21: c.regs = 168; taps_gather = 1.16; taps_lat = 1.07; c.eff_sat = 0.50; c.t_lat_us = 0.489; c.t_round_us = 2.24; c.gather_cycles = 36.3; tap_gather = 0.845; c.split_c0 = 2.37; break;
            case 22: c.regs = 256; taps_gather = 1.24; taps_lat = 1.16; c.eff_sat = 0.615; c.t_lat_us = 0.772; c.t_round_us = 2.84; c.gather_cycles = 38.5; tap_gather = 0.488; c.split_c0 = 2.44; break;
            default: c.regs = 256; taps_gather = 0.89; taps_lat = 0.98; c.eff_sat = 0.659; c.t_lat_us = 0.361; c.t_round_us = 6.5; c.gather_cycles = 67.3; tap_gather = 0.99; c.split_c0 = 0.45; break;
            }
        }
        // 1x1 filters without padding: the channel rides in the instruction's uniform offset and the
        // lanes read a contiguous run of pixels (stride 1); with a stride the lanes' addresses are
        // spread over several times the cache lines and the loads cost what gathered ones do
        if (point) {
            if (q.stride == 1) c.gather_cycles *= point_gather;
        } else if (cfg.layout == 2 && q.stride == 1) {
            // tap by tap over the [K][R][S][C] filter copy: one tap per stage, so the validity bit and
            // the distance are worked out per stage and not per element
            // (with a stride the lanes' addresses spread over twice the cache lines and the cost of
            // the load is in the memory pipeline, which the cheaper addressing does not touch)
            c.gather_cycles *= tap_gather;
        } else if (split && gather_table_fits(q, cfg.bk)) {
            c.gather_cycles *= table_gather;
        } else if (q.K <= 64) {   // one row of tiles
            c.gather_cycles *= taps_gather;
            c.t_lat_us *= taps_lat;
        }
        // and splitting the reduction gains less there than the fit to mostly unstrided layers says: 128 -> 128 3x3/2
        // on 56x56, batch 32, tile 128x128: two parts 66.9 us, whole tiles 60.1 (stride 1, 28x28: 56.0 and 59.4)
        if (split && cfg.layout == 2 && q.stride > 1) c.split_c0 += 3;
        if (c.split_c1 == 0) c.split_c1 = 0.1;   // scratch tiles, as in the patch kernel
    }
    Shape s = conv_shape(q, cfg.algo, cfg.bn, std::max(2, cfg.cb));
    model(s, c, r);
}

// bfloat16 patch kernel; q.C counts units of eight channels.  Same round-by-round timing as the
// fp32 kernels with the bf16 instruction's rate (a 32x32x16 step takes 32 cycles).  The stage
// efficiency is low because every step needs two 16-byte operand reads per lane from LDS, which
// the LDS cannot deliver at the matrix cores' pace; constants fitted to a sweep of the family on
// the ResNet-50-shaped suite at batch 64.
double model_conv_bf16(const ConvProblem &q, const polydl_tile_cfg &cfg, int threads)
{
    const double RS = (double)q.R * q.S;
    const int cb = q.C == 1 ? 1 : std::max(2, cfg.cb);
    const double mb = cfg.wm / 32.0, nb = cfg.wn / 32.0, waves_per_wg = threads / 64.0;
    const double Ng = (double)q.N * q.P * q.Q;
    const double tiles = std::ceil((double)q.K / cfg.bm) * std::ceil(Ng / cfg.bn);
    const double RSp = (double)patch_rows_per_stage(q) * q.S;
    const double nstages = std::ceil((double)q.C / cb) * (q.R / patch_rows_per_stage(q));
    const double per_split = std::ceil(nstages / std::max(1, cfg.split_k));
    const double parts = std::ceil(nstages / per_split);
    const double wp = q.S == 1 ? q.Q : q.W + 2 * q.pad;
    // the kernel's stage buffers: filter rows of odd pitch, both operands rounded up to whole
    // passes of the workgroup
    const double lda = (double)(((int)(cb * RSp) + 1) | 1);
    const double stage_units = std::ceil(cfg.bm * lda / threads) * threads +
                               std::ceil(cb * conv_patch_rows(q, cfg.bn) * wp / threads) * threads;
    const double lds_bytes = ((per_split > 1 ? 2.0 : 1.0) * stage_units + 64) * 16;
    const int waves_per_simd = mb * nb == 4 ? 3 : 4;   // from the kernels' register counts
    const double occ = std::max(1.0, std::min(std::floor(waves_per_simd * kSimdsPerCU / waves_per_wg),
                                              std::floor(160.0 * 1024 / lds_bytes)));
    // per wave tile: stage efficiency, per-round latency, stage latency floor, bytes per microsecond a
    // CU stages into LDS, split cost per MB of parts
    double eff = 0.25, t_round = 3.0, t_lat = 0.8, rate = 60000.0, c1 = 0.1;
    if (mb * nb == 2) { eff = 0.4; t_round = 4.0; c1 = 0.2; }
    else if (mb * nb == 4) { eff = 0.4; t_round = 4.0; t_lat = 0.4; rate = 31000.0; c1 = 0.4; }
    // matrix instructions of a stage per accumulator block: one per tap and pair of units; a
    // reduction of a single unit takes two taps per instruction instead
    const double steps = q.C == 1 ? std::ceil(RSp / 2.0) : std::ceil(cb / 2.0) * RSp;
    const double t_stage = std::max(steps * mb * nb * 32.0 * std::ceil(waves_per_wg / kSimdsPerCU) /
                                        kClockHz * 1e6 / eff,
                                    (cfg.bm * cb * RSp + cb * conv_patch_rows(q, cfg.bn) * wp) * 16.0 / rate);
    const double per_cu = tiles * parts / kCUs;
    const double full_rounds = std::floor(per_cu / occ), rest = per_cu - full_rounds * occ;
    auto round_us = [&](double n) { return t_round + per_split * std::max(n * t_stage, t_lat); };
    double t = full_rounds * round_us(occ) + (rest > 1e-9 ? round_us(std::ceil(rest - 1e-9)) : 0.0);
    const double d_bytes = (double)q.N * q.K * q.P * q.Q * 4;
    const double mem_bytes = (double)q.N * q.C * 8 * q.H * q.W * 2 + (double)q.K * q.C * 8 * RS * 2 + d_bytes;
    t = 5.0 + std::max(t, mem_bytes / 6000.0 * 1e-3 + 2.0);
    if (parts > 1) t += c1 * parts * d_bytes * 1e-6;
    return t;
}

void model_sgemm(const SgemmProblem &q, const polydl_tile_cfg &cfg, int threads, polydl_model_report *r)
{
    Shape s;
    s.Mg = q.M; s.Ng = q.N; s.Kg = std::ceil((double)q.K / cfg.bk) * cfg.bk;
    s.a_bytes = (double)q.M * q.K * 4;
    s.b_bytes = (double)q.K * q.N * 4;
    s.d_bytes = 2.0 * q.M * q.N * 4;                                       // C is read and written
    s.b_tile_bytes = (double)cfg.bn * q.K * 4;
    Cand c;
    c.bm = cfg.bm; c.bn = cfg.bn; c.wm = cfg.wm; c.wn = cfg.wn; c.threads = threads;
    c.split_k = std::max(1, cfg.split_k);
    c.steps_per_stage = cfg.bk / 2.0;
    c.lds_bytes = 2.0 * (cfg.bm * (cfg.bk + 4) + cfg.bk * (cfg.bn + 4)) * 4;
    c.loop_eff = 0.84;
    c.wg_overhead_cycles = 3000;
    c.kernel_fixed_us = 6.0;
    // from the kernels' register counts (the eight-block wave tiles are held to 256 registers)
    c.max_waves_per_simd = (cfg.wm * cfg.wn > 64 * 64) ? 2 : ((cfg.wm * cfg.wn == 64 * 64) ? 3 : 4);
    if (q.beta != 0.f && cfg.wm * cfg.wn >= 64 * 64) c.read_overhead = cfg.wm * cfg.wn > 64 * 64 ? 8844 : 7789;
    double part_rate = 1.0, part_us = 0.4, parts_us = 0.0;
    if (split_products(cfg.bk, cfg.wm, cfg.wn) && q.K >= kSgemmSplitMinReduction) {
        // Fitted to sweeps of 1142 sizes, 64 .. 4096 by 64 .. 4096 by 8 .. 32768, odd ones and accumulated ones among them:
        // the picks run within 1 % of the sweep's best on average, 24 % at worst (64x64x8).  The smaller the wave tile, the more
        // splitting and the more LDS reads per matrix instruction; 512 threads split a 256x128 tile's operands
        // once for twice the outputs.  Large tiles pay for their epilogue, most of all where C is read: few
        // workgroups then wait for row after row (1418x747x39, accumulated: 64x64 10.6 us, 128x128 22).
        const int blocks = cfg.wm * cfg.wn / 1024;
        const int k = blocks == 1 ? 0 : blocks == 2 ? 1 : threads == 512 ? 3 : 2;
        static const double kEff[] = {0.339, 0.449, 0.595, 0.648}, kStore[] = {1012, 1942, 9413, 4443}, kRead[] = {2110, 5074, 12511, 10714};
        c.split = true;
        c.split_eff = kEff[k];
        c.split_overhead = kStore[k];
        c.read_overhead = q.beta != 0.f ? kRead[k] : 0;
        c.max_waves_per_simd = blocks == 1 ? 4 : blocks == 2 ? 3 : 2;
        c.lds_bytes = split_lds_bytes(cfg.bm, cfg.bn);
        // the last part of a tile adds all parts alone, at what one compute unit can read (60 GB/s)
        part_rate = 0.19; part_us = 0.215; parts_us = 1.36 + cfg.split_k * (double)cfg.bm * cfg.bn * 4 / 59.6 * 1e-3;
    }
    model(s, c, r);
    if (cfg.split_k > 1) {   // every part writes its tile to scratch once, the last one reads them all back
        // plus the hand-over itself (store, count, read back), which no amount of bandwidth shortens
        r->fixed_us = c.kernel_fixed_us + 2.0 * part_rate * cfg.split_k * (double)q.M * q.N * 4 / kHbmGBs * 1e-3 +
                      part_us * (cfg.split_k - 1) + parts_us;
        r->predicted_us = std::max(r->mfma_us, r->mem_us) + r->fixed_us;
    }
}

static const int kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16};

// Pointwise kernel (filter resident in LDS, pixels loaded straight into registers): a unit is
// 64 pixels x 32 output channels, 12 bfloat16 matrix instructions per 16 channels; units are dealt to the waves in
// equal runs, so the busiest SIMD runs ceil(units / SIMDs) of them one after another.  The tensors
// are streamed once.
void model_conv_point(const ConvProblem &q, polydl_model_report *r)
{
    std::memset(r, 0, sizeof(*r));
    uint32_t units, wgs;
    conv_point_shape(q, kCUs, &units, &wgs);
    const double pixels = (double)q.N * q.H * q.W;
    const double in_bytes = pixels * q.C * 4, out_bytes = pixels * q.K * 4, wt_bytes = (double)q.K * q.C * 4;
    const double unit_us = (q.C / 16.0) * 12.0 * 32.0 / kClockHz * 1e6;
    const double per_simd = std::ceil((double)units / (kCUs * kSimdsPerCU));
    r->mfma_us = per_simd * unit_us / 0.85;
    // measured on 64 -> 256 channels at 56 x 56, batch 32 and 64 (back-to-back launches on the same buffers):
    // the time follows the bytes written, at 4.3 TB/s; the input, re-read from the last-level cache, hardly shows
    r->mem_us = (in_bytes + wt_bytes) / 20000.0 * 1e-3 + out_bytes / 4300.0 * 1e-3;
    r->fixed_us = 7.0;                               // launch, filling LDS with the filter, first loads, last stores
    r->predicted_us = std::max(r->mfma_us, r->mem_us) + r->fixed_us;
    r->workgroups = (int)wgs;
    r->simd_load = per_simd;
    // reuses: accumulators of a unit (registers); the pixel registers reused by the channel groups;
    // the filter in LDS reused by every unit (read once per unit); the tensors themselves
    const double ws[4] = {32.0 * 64 * 4, 64.0 * q.C * 4, wt_bytes, in_bytes + out_bytes + wt_bytes};
    const double moved[4] = {0, 0, (double)units * 32.0 * q.C * 4, in_bytes + out_bytes + wt_bytes};
    double sizes[4], weights[4];
    for (int i = 0; i < 4; ++i) { sizes[i] = kLevels[i].capacity; weights[i] = 1.0 / kLevels[i].gbytes_per_s; }
    int placed[4];
    bucket_placed(4, ws, 4, sizes, r->level_bytes, &r->mem_bytes, placed);
    r->eq1_cost = reuse_cost(4, r->level_bytes, r->mem_bytes, weights, 1.0 / kHbmGBs);
    r->n_ws = 4;
    for (int i = 0; i < 4; ++i) { r->ws[i] = ws[i]; r->ws_level[i] = placed[i]; r->ws_traffic[i] = moved[i]; }
}

// First-layer kernel (split filter resident in LDS, pixels gathered straight into registers): units of 64 pixels, dealt evenly to
// the waves, two of which share a SIMD.  Fitted to 1916 launches of 24 .. 384 reduction rows and 1536 .. 40000 units, operands in the
// cache: 11 % off in the mean, 25 % below to 14 % above for eight of ten.
void model_conv_thin(const ConvProblem &q, polydl_model_report *r)
{
    std::memset(r, 0, sizeof(*r));
    const double Kg = (double)q.C * q.R * q.S, steps = std::ceil(Kg / 32) * 2, pixels = (double)q.N * q.P * q.Q;
    const double units = std::ceil(pixels / 64), waves = std::min(kCUs * 8.0, std::ceil(units / 8) * 8);
    const double in_bytes = (double)q.N * q.C * q.H * q.W * 4, out_bytes = pixels * q.K * 4, wt_bytes = q.K * Kg * 4;
    // a last round of at most half the waves finds the SIMDs to itself
    const double full = std::floor(units / waves), rest = units / waves - full;
    const double rounds = full + (rest <= 0 ? 0.0 : rest <= 0.5 ? 0.26 : 1.0);
    r->mfma_us = rounds * (steps * 1.36 + 2.6 + 0.4 * q.K / 64.0);
    r->mem_us = in_bytes / 5400.0 * 1e-3 + out_bytes / 3460.0 * 1e-3;
    r->fixed_us = 5.6;                               // launch, splitting the filter into LDS, first loads, last stores
    r->predicted_us = std::max(r->mfma_us, r->mem_us) + r->fixed_us;
    r->workgroups = (int)(waves / 8);
    r->simd_load = std::ceil(units / (waves / 2));
    // reuses: accumulators of a unit; its pixels' values, reused by the channels; the filter's planes in LDS, read by every unit;
    // the tensors themselves
    const double planes = steps * 16 * 64 * 6;
    const double ws[4] = {2 * 64.0 * 64 * 4, 64.0 * Kg * 4, planes, in_bytes + out_bytes + wt_bytes};
    const double moved[4] = {0, units * 64.0 * Kg * 4, units * planes, in_bytes + out_bytes + wt_bytes};
    double sizes[4], weights[4];
    for (int i = 0; i < 4; ++i) { sizes[i] = kLevels[i].capacity; weights[i] = 1.0 / kLevels[i].gbytes_per_s; }
    int placed[4];
    bucket_placed(4, ws, 4, sizes, r->level_bytes, &r->mem_bytes, placed);
    r->eq1_cost = reuse_cost(4, r->level_bytes, r->mem_bytes, weights, 1.0 / kHbmGBs);
    r->n_ws = 4;
    for (int i = 0; i < 4; ++i) { r->ws[i] = ws[i]; r->ws_level[i] = placed[i]; r->ws_traffic[i] = moved[i]; }
}

// ---- small problems: single waves (wave_core.hpp) --------------------------------------------------
// Predicted microseconds of tiles of 64x64 shared by eight waves (one workgroup on a compute unit) or four (two), and of 32x32 (two).
// Fitted to 30684 launches (2700 drawn problems of 2e6 .. 3e10 flops, 1 .. 16 parts): 7.6 % off in the mean, 15 % in 95 of 100.  A step
// costs a workgroup 0.52 (32x32) .. 1.2 us; gathered operands cost up to 1.7 times that, and up to 1.8 us before the first step.
// bfloat16 (a step is four units of eight channels): 7969 launches of 1000 drawn layers of 5e6 .. 3e10 flops, 9 % off in the mean; 64x64 shared by
// four waves: 11162 launches of 3000 layers of 5e6 .. 6e10, 7.6 % off.
enum WaveLoads { WAVE_ROWS, WAVE_POINT, WAVE_POINT_STRIDED, WAVE_TAP, WAVE_TAP_STRIDED, WAVE_TAPS, WAVE_TAPS_STRIDED,
                 WAVE_BF16_POINT, WAVE_BF16_POINT_STRIDED, WAVE_BF16_TAPS, WAVE_BF16_TAPS_STRIDED };
// step1, step2: one, two workgroups on a compute unit; most: weight of the longest wave's steps against the mean; whole: of whole rounds
struct WaveFit { double launch, round, step1, step2, parts, part, most, whole; };
static const WaveFit kWave32 = {1.6, 2.43, 0.519, 1.127, 1.24, 0.19, 0.28, 0.37}, kWave64 = {0.9, 4.3, 1.20, 0, 1.66, 0.25, 0.1, 1},
                     kWave64x4 = {1.2, 3.87, 0.72, 1.32, 1.78, 0.30, 0.73, 0.48}, kWaveBf16_32 = {2.0, 2.4, 0.168, 0.395, 1.42, 0.19, 1, 0.4},
                     kWaveBf16_64 = {2.1, 3.7, 0.381, 0, 1.77, 0.23, 0.33, 1}, kWaveBf16_64x4 = {1.86, 2.99, 0.253, 0.56, 1.74, 0.295, 1, 0.60};
// steps_us (may be null): the time of the steps alone
static double wave_us(int tile, int waves, int parts, double tiles, double steps, WaveLoads loads, double out_bytes, double *steps_us = nullptr)
{
    // the last four: bfloat16 on four waves
    static const double per_step[] = {1, 1.26, 1.66, 1.08, 1.27, 1.14, 1.23, 1, 1.53, 1.39, 1.59, 1, 1.62, 1.15, 1.27};
    static const double before[] = {0, 1.00, 0.83, 1.23, 1.30, 1.53, 1.79, 0, -0.27, -0.27, -0.60, 0, -0.27, -0.05, -0.38};
    const bool bf16 = loads >= WAVE_BF16_POINT;
    const int kind = loads + (bf16 && waves == 4 ? 4 : 0);
    const WaveFit &f = bf16 ? (tile == 32 ? kWaveBf16_32 : waves == 4 ? kWaveBf16_64x4 : kWaveBf16_64) : tile == 32 ? kWave32 : waves == 4 ? kWave64x4 : kWave64;
    const double mean = std::ceil(steps / parts) / waves, n = (f.most * std::ceil(mean) + (1 - f.most) * mean) * per_step[kind];
    const double wgs = tiles * parts, cus = kCUs, full = wgs / (f.step2 > 0 ? 2 * cus : cus);
    const double rounds = full <= 1 ? 1 : f.whole * std::ceil(full) + (1 - f.whole) * full;
    // one round if two workgroups fit a compute unit and there is no more than one for each
    const bool pairs = f.step2 > 0 && wgs > cus;
    const double times = f.step2 > 0 && !pairs ? 1 : rounds, each = n * (pairs ? f.step2 : f.step1);
    if (steps_us) *steps_us = times * each;
    return before[kind] + out_bytes / 4.0e6 + f.launch + (parts > 1 ? f.parts + f.part * parts : 0) + times * (f.round + each);
}
static WaveLoads wave_loads(const ConvProblem &q, int layout)
{
    const int strided = q.stride > 1;
    if (q.R == 1 && q.S == 1 && q.pad == 0) return strided ? WAVE_POINT_STRIDED : WAVE_POINT;
    if (layout == 2) return strided ? WAVE_TAP_STRIDED : WAVE_TAP;
    return strided ? WAVE_TAPS_STRIDED : WAVE_TAPS;
}
// Products: the least time of what the XCDs bring in, the operands from memory and what several of them read once more from the last-level cache.
// Each takes a run of tiles (WaveOrder) and reads the panels these touch once; row_bytes: of a row's reduction.  Of 3500 drawn products of more
// than 8 MB the larger of this and the formula above is 17 % off in the mean, the formula alone 29 %, 2.3 times too low at
// worst (105x236x466615).
static double wave_panels_us(int tile, double M, double N, double row_bytes)
{
    const double tm = std::ceil(M / tile), tn = std::ceil(N / tile), run = std::ceil(tm * tn / 8), rows = std::min({run, tm, 8.0});
    const double once = M + N, all = std::min(8.0, tm * tn) * (rows * M / tm + std::ceil(run / rows) * N / tn);
    return (once / 5.0e6 + std::max(0.0, all - once) / 4.5e6) * row_bytes;
}
// The best of the tiles and 1 .. 16 parts, if it is predicted below `limit`, for tiles of 64x64 `limit64`.  row_bytes: of products,
// 0 for convolutions; a product's panels have to be predicted below panels_limit.
template <class Fits>
static bool wave_best(double M, double N, double steps, WaveLoads loads, int layout, double limit, double limit64, bool no_scratch, const ScratchArena *arena,
                      Fits &&fits, polydl_tile_cfg *cfg, double row_bytes = 0, double panels_limit = 0)
{
    static const int kParts[] = {1, 2, 3, 4, 6, 8, 12, 16}, kTiles[][2] = {{32, 8}, {64, 8}, {64, 4}};
    const double cus = kCUs;
    bool found = false;
    for (const int (&tw)[2] : kTiles) {
        const int tile = tw[0], waves = tw[1];
        if (!fits(tile) || (row_bytes > 0 && wave_panels_us(tile, M, N, row_bytes) >= panels_limit)) continue;
        const double tiles = std::ceil(M / tile) * std::ceil(N / tile);
        // a handful of tiles of a few steps each: waves without work
        if (tile == 32 && steps < kWavesPerTile && tiles < 16) return false;
        if (tiles > 4096) continue;
        if (tile == 64) limit = std::min(limit, limit64);
        for (int parts : kParts) {
            if (parts > 1 && (no_scratch || parts * 4 > steps || tiles * parts > (tile == 64 && waves == 8 ? 2 : 4) * cus)) break;
            if (parts > 1 && arena && (tiles * parts * tile * tile * 4 > arena->partial_bytes || tiles > arena->ncounters)) break;
            double us = wave_us(tile, waves, parts, tiles, steps, loads, M * N * 4);
            // parts of a reduction of few tiles are 2 .. 3 % better than the formula has it
            if (parts == 1 && tiles <= 64) us *= 1.02;
            // in bfloat16 the four waves have to be well below the eight: without this one in fifty layers is 3 % slower than on those
            if (waves == 4 && loads >= WAVE_BF16_POINT) us *= 1.03;
            if (us >= limit) continue;
            limit = us;
            *cfg = wave_cfg(tile, waves, parts, layout);
            found = true;
        }
    }
    return found;
}

// Whether a small problem goes to single waves, given its pick's prediction: a margin for what the two predictions are off, and further down lower
// ones where one of them is further off.  Drawn over 1 .. 4096 channels, 1 .. 224 pixels a side, batches of 1 .. 128 and 2e6 .. 4e10 flops, 12351 of
// 22501 layers in the KCRS order go there and take 0.70 of the pick's time in sum, 70 of them more than 3 % longer; with the filter's copy 12539 of
// 22480, 0.72, 110; 1x1 layers 13260 of 44326, 0.71, 82; products of up to 8192 x 8192 x 200000 14217 of 19353, 0.60, 29.  The lower margins lie where
// the mean of a class comes to the pick's time, or where many of it take much longer.
// Picks of more than 40 us gain little and are mispredicted more often.  Convolutions of
// fewer than 128 reduction rows run on the fp32 instruction otherwise and are predicted too high, by up to 1.6.
// Reductions of fewer steps than there are waves have a rounding per step and those of the meeting, which a staged tile sums in one accumulator:
// against 64 bits they are further off, products of 32, 40, 64, 96 by 14, 22, 8, 2 %; from 112 on nearer (128: 5 %, 256: 5 .. 26 %).  Staged
// tiles that split the reduction are the more exact up to 160 (144 in three parts: by 3 %; 192: the waves by 1 %).
static bool wave_exact(int64_t Kg, const polydl_tile_cfg &pick) { return Kg >= (pick.split_k > 1 ? 192 : 112); }
static double wave_limit(double pick_us, bool short_rows) { return pick_us * (short_rows ? 0.6 : pick_us <= 40 ? 0.9 : 0.83); }
// Cache lines under the values of one reduction row that 64 neighbouring pixels of the output read, unpadded.
static double row_lines(const ConvProblem &q)
{
    const double PQ = (double)q.P * q.Q, pixels = std::min(64.0, q.N * PQ);
    return std::min(pixels / q.Q * (1 + q.Q * q.stride / 32.0), std::max(1.0, pixels / PQ) * (1 + (double)q.H * q.W / 32));
}
// Unsplit picks of 1x1 layers on the gather kernel are predicted too high: they take 0.76 of it at 128 rows, 0.86 at 500, on the fp32
// instruction 0.72 .. 0.8, strided ones into at most 64 channels down to 0.58, and there the waves' tiles, one row of them, take up to 1.5 times
// what they are predicted.  With the margins of other layers 42 of 74 strided ones into up to 64 channels were slower than their pick, by up to 31 %
// (128 -> 64 on 56x45, batch 32: 13.1 us against 10.2), 40 of 183 into more, by up to 13 %, and 10 of 14 unstrided ones of 128 rows into
// up to 64, by up to 17 %; the three margins lie where layers drawn anew
// come to the pick's time: strided ones into up to 64 above 0.5 (1300: 1.02), others above 0.8 (2130: 1.02), unstrided ones above 0.85 (1936: 0.99).
bool conv_wave_pick(const ConvProblem &q, double pick_us, bool no_scratch, polydl_tile_cfg *cfg)
{
    const int64_t Kg = (int64_t)q.C * q.R * q.S;
    if (!wave_exact(Kg, *cfg)) return false;
    const bool point_pick = cfg->algo == 0 && cfg->split_k <= 1 && q.R == 1 && q.S == 1 && q.pad == 0;
    const int layout = q.has_tap && gather_tap_major_fits(q, 16) ? 2 : 0;
    double limit = wave_limit(pick_us, Kg < kSplitMinReduction || (point_pick && !split_pays(q.K, 1, Kg)));
    if (point_pick) limit = std::min(limit, (q.stride == 1 ? 0.84 : q.K > 64 ? 0.8 : 0.5) * pick_us);
    // up to 64 channels in the KCRS order: the gather kernel's 64x128 tiles take 0.75 .. 0.82 of their prediction (1019 -> 64 3x3 on 28x28, batch
    // 32: 212 us; waves 230).  74 of 987 such layers were slower on the waves, by up to 10 %; 7 of the 672 that still go there, by up to 9 %
    if (layout == 0 && q.R * q.S > 1 && q.K <= 64 && cfg->algo == 0 && cfg->bn == 128) limit = std::min(limit, 0.76 * pick_us);
    // strided layers tap by tap: a wave's loads spread over twice the cache lines, and a tile's waves come back to a line a whole tap later,
    // when many channels have passed and it is gone: up to 2.5 times what they are predicted, 10 times on inputs beyond the caches (512 -> 64 7x7
    // on 14x18, batch 64: 112 us, waves 214; 3264 -> 23 4x4 on 21x9, batch 74: 148 and 422).  384 channels and more on inputs beyond 16 MB come to
    // 0.86 .. 1.0 of the pick's time from 0.5 on, one in nine more than 10 % slower, by up to 191 %; other layers into more than 64 channels to 0.98 above 0.77;
    // into fewer they take 0.9 up to 0.85, from 384 channels 0.89 at 0.65 .. 0.7 (4000 layers drawn among those above these or lower margins)
    const double in_bytes = 4.0 * q.N * q.C * q.H * q.W, operands = in_bytes + 4.0 * q.K * Kg;
    if (layout == 2 && q.stride > 1) {
        const bool deep = q.C >= 384;
        const double margin = deep && in_bytes > 16e6 ? 0.5 : q.C > 1024 && operands > 64e6 ? 0.62 : q.K > 64 ? 0.77 : deep && pick_us > 20 ? 0.72 : 0.83;
        limit = std::min(limit, margin * pick_us);
    }
    // Loads that spread over many lines, and inputs beyond 256 MB, cost the waves up to three times what they are predicted.  In the KCRS order they
    // are even from 23 lines on above 0.8 (361 drawn layers: 1.01 of the pick's time, 38 % slower; 0.75 .. 0.8: 0.87, 10 %), large inputs
    // above 0.7 (70: 0.97, 20 slower); with the copy from 16 lines on above 0.75 (220: 0.97, 31 % slower; 0.65 .. 0.75: 0.91, 15 %), operands beyond 64 MB
    // above 0.8 (110: 0.92).  The margins for lines lie lower, where the slowest begin: single layers take up to 1.6 times as long
    const bool point = q.R == 1 && q.S == 1 && q.pad == 0;
    const double lines = row_lines(q);
    if (lines >= (layout == 0 ? 23 : 16)) limit = std::min(limit, (layout == 0 ? 0.75 : 0.66) * pick_us);
    if (layout == 0 ? in_bytes > 256e6 : operands > 64e6) limit = std::min(limit, (layout == 0 ? 0.7 : 0.8) * pick_us);
    // Strided 1x1 layers whose pick splits gain nothing on tiles of 64x64 above 0.85 (1007: 0.99, 23 % slower; 0.8 .. 0.85: 0.9), nor at all above 0.7
    // on inputs beyond 64 MB (42: 1.0, 19 slower); unsplit ones on inputs beyond 32 MB not above 0.75, at stride 3 not above 0.4 (31: 0.98, 10 slower,
    // and 106: 0.96, 42, by up to 26 %, 128 -> 128 on 68x68, batch 53, 18.4 us and 23.1)
    double limit64 = pick_us;
    if (point && q.stride > 1) {
        const bool split = cfg->split_k > 1;
        if (split) limit64 = (in_bytes > 64e6 ? 0.6 : 0.85) * pick_us;
        if (in_bytes > (split ? 64e6 : 32e6)) limit = std::min(limit, (split ? 0.7 : q.stride == 2 ? 0.75 : 0.4) * pick_us);
    }
    return wave_best(q.K, (double)q.N * q.P * q.Q, std::ceil(Kg / 16.0), wave_loads(q, layout), layout, limit, limit64, no_scratch, q.arena,
                     [&](int tile) { return conv_wave_fits(q, tile); }, cfg);
}
bool sgemm_wave_pick(const SgemmProblem &q, double pick_us, bool no_scratch, polydl_tile_cfg *cfg)
{
    if (!wave_exact(q.K, *cfg)) return false;
    // Long reductions: picks of 48 parts and more take 0.7 of their prediction, and neither formula knows how much of the panels the caches keep.
    // Beyond 16384 products above 0.6 (picks of fewer parts; 1138 drawn: 0.98 of the pick's time, 29 % slower) and 0.5 (433: 1.14, 64 %; 105x236x466615
    // 283 us, waves 656) are even or worse, and so are those whose panels take more than 0.9 of the pick's prediction (330: 1.02; 0.8 .. 0.9: 0.92, 22 %
    // slower); up to 16384 those below 0.85 take 0.82 .. 0.9 and one in fifty is slower
    const bool longer = q.K > 16384;
    const double limit = std::min(wave_limit(pick_us, false), !longer ? pick_us : cfg->split_k >= 48 ? 0.45 * pick_us : 0.58 * pick_us);
    return wave_best(q.M, q.N, std::ceil(q.K / 16.0), WAVE_ROWS, 0, limit, limit, no_scratch, q.arena,
                     [&](int tile) { return sgemm_wave_fits(q, tile); }, cfg, 4.0 * q.K, (longer ? 0.8 : 0.85) * pick_us);
}

// bfloat16, q.C units of eight channels.  The margins are the staged model's: of 3000 drawn layers of 5e6 .. 6e10 flops the picks of 1x1 ones take
// 0.82 .. 0.92 of their prediction, of others 1.02 .. 1.17, but 0.8 where a reduction of up to 20 steps is one stage; beyond 256 steps both are off.  Over
// the ranges above 16035 of 24283 layers go there and take 0.62 of the pick's time in sum, 91 of them more than 3 % longer; 1x1 layers 17132 of 38410,
// 0.64, 43.  Up to eight units a row leave most waves without a
// step; picks predicted at the floor of their model (8.8 us) take 5 us and more, which the larger tile does not undercut.
// Where the margins lie, of 17000 layers drawn among those above lower ones: picks that do not split take 0.8 .. 0.9 of their prediction at 36 steps
// (128 input channels 3x3), and strided layers of more than 40 us cost the waves 1.2 .. 1.4 times theirs: above 0.9, and above 0.85 where a
// pick of up to 48 steps takes more than 18 us, they come to the pick's time (803 -> 256 3x3/2 on 28x28, batch 36: 50 us, waves 63).
// Two and three steps a row (8 -> 8 3x3), whose pick takes 0.55 .. 0.7 of the model's floor: 0.98 at 0.5 .. 0.55, 1.05 .. 1.11 above; four and five: 0.94 at
// 0.6 .. 0.65, 1.0 above.  Operands beyond 64 MB take the waves up to 2.5 times what they are predicted, filters beyond 64 MB above 0.72: 1.0 (263, 32 %
// more than 10 % slower), more than 1024 channels 0.85 (652, 19 %), others 0.84 up to 0.9 (1269, 4 %), 0.95 above; strided layers with filters beyond 20 MB
// of more than 1024 channels 0.88 above 0.7 (362, 23 %; 2513 -> 743 3x3/3 on 100x3, batch 18: 53 us, waves 98), of fewer 0.76 (730, 4 %).  1x1 layers of more
// than 15 us and 64 steps: 0.92 at 0.6 .. 0.65 (13 %), 1.0 above; strided ones of up to five steps on inputs beyond 16 MB 0.92 at 0.5 .. 0.55, 0.97 above.
static WaveLoads wave_bf16_loads(const ConvProblem &q)
{
    const bool strided = q.stride > 1;
    if (q.R == 1 && q.S == 1) return strided ? WAVE_BF16_POINT_STRIDED : WAVE_BF16_POINT;
    return strided ? WAVE_BF16_TAPS_STRIDED : WAVE_BF16_TAPS;
}
bool conv_wave_bf16_pick(const ConvProblem &q, double pick_us, bool no_scratch, polydl_tile_cfg *cfg)
{
    const int64_t units = (int64_t)q.C * q.R * q.S;
    if (units <= 8) return false;
    const double steps = std::ceil(units / 4.0);
    const bool unsplit = cfg->split_k <= 1, point = q.R == 1 && q.S == 1, strided = q.stride > 1, deep = q.C > 128;
    const double in_bytes = 16.0 * q.N * q.C * q.H * q.W, filter_bytes = 16.0 * units * q.K;
    double margin = point           ? (pick_us > 15 && units > 256 ? 0.6 : 0.72)
                    : steps < 4     ? 0.52
                    : steps < 6     ? 0.65
                    : steps < 20    ? (q.K <= 32 ? 0.76 : 0.8)
                    : steps > 256   ? 0.88
                    : !unsplit      ? 0.92
                    : !strided      ? 0.9
                    : pick_us > 40  ? 0.9
                                    : steps <= 48 && pick_us > 18 ? 0.85 : 0.92;
    if (strided && !point && deep && filter_bytes > 20e6) margin = std::min(margin, 0.7);
    if (strided && point && unsplit && steps <= 5 && in_bytes > 16e6) margin = 0.5;
    if (pick_us > 20 && in_bytes + filter_bytes > 64e6) margin = std::min(margin, deep || filter_bytes > 64e6 ? 0.72 : 0.88);
    const double limit = margin * pick_us;
    return wave_best(q.K, (double)q.N * q.P * q.Q, steps, wave_bf16_loads(q), 0, limit, pick_us < 9.5 ? 0.73 * pick_us : limit, no_scratch,
                     q.arena, [&](int tile) { return conv_wave_bf16_fits(q, tile); }, cfg);
}

double model_conv_wave_bf16(const ConvProblem &q, const polydl_tile_cfg &cfg)
{
    const double M = q.K, N = (double)q.N * q.P * q.Q;
    return wave_us(cfg.bm, wave_cfg_waves(cfg), std::max(1, cfg.split_k), std::ceil(M / cfg.bm) * std::ceil(N / cfg.bm), std::ceil(q.C * q.R * q.S / 4.0),
                   wave_bf16_loads(q), M * N * 4);
}

static void model_wave(double M, double N, double Kg, WaveLoads loads, double in_bytes, const polydl_tile_cfg &cfg, polydl_model_report *r)
{
    std::memset(r, 0, sizeof(*r));
    const double t = cfg.bm, tiles = std::ceil(M / t) * std::ceil(N / t), parts = std::max(1, cfg.split_k);
    r->predicted_us = wave_us(cfg.bm, wave_cfg_waves(cfg), (int)parts, tiles, std::ceil(Kg / 16), loads, M * N * 4, &r->mfma_us);
    r->mem_us = (in_bytes + M * Kg * 4 + M * N * 4) / kHbmGBs * 1e-3;
    // launch, rounds, first loads, hand-over and stores: what neither the steps nor the tensors' bytes take
    r->fixed_us = std::max(0.0, r->predicted_us - std::max(r->mfma_us, r->mem_us));
    r->workgroups = (int)std::min(tiles * parts, 2e9);
    r->simd_load = std::ceil(tiles * parts / kCUs) * wave_cfg_waves(cfg) / kSimdsPerCU;
    // reuses: accumulators over a wave's steps; a step's operands, every row with every column; the operands by the tiles; the tensors
    const double all = in_bytes + M * Kg * 4 + M * N * 4;
    const double ws[4] = {2 * t * t * 4, 2 * t * 16 * 4, 2 * t * Kg * 4, all};
    const double moved[4] = {0, tiles * 2 * t * Kg * 4, tiles * 2 * t * Kg * 4, all};
    double sizes[4], weights[4];
    for (int i = 0; i < 4; ++i) { sizes[i] = kLevels[i].capacity; weights[i] = 1.0 / kLevels[i].gbytes_per_s; }
    int placed[4];
    bucket_placed(4, ws, 4, sizes, r->level_bytes, &r->mem_bytes, placed);
    r->eq1_cost = reuse_cost(4, r->level_bytes, r->mem_bytes, weights, 1.0 / kHbmGBs);
    r->n_ws = 4;
    for (int i = 0; i < 4; ++i) { r->ws[i] = ws[i]; r->ws_level[i] = placed[i]; r->ws_traffic[i] = moved[i]; }
}

void model_conv_wave(const ConvProblem &q, const polydl_tile_cfg &cfg, polydl_model_report *r)
{
    model_wave(q.K, (double)q.N * q.P * q.Q, (double)q.C * q.R * q.S, wave_loads(q, cfg.layout), (double)q.N * q.C * q.H * q.W * 4, cfg, r);
}
void model_sgemm_wave(const SgemmProblem &q, const polydl_tile_cfg &cfg, polydl_model_report *r)
{
    model_wave(q.M, q.N, q.K, WAVE_ROWS, (double)q.K * q.N * 4, cfg, r);
}

void conv_candidates(const ConvProblem &q, std::vector<ConvCandidate> *out)
{
    out->clear();
    ConvCandidate cand;
    if (conv_point_fits(q)) {
        cand.cfg = conv_point_cfg();
        model_conv_point(q, &cand.rep);
        out->push_back(cand);
    }
    const int cpad = (q.C + 1) & ~1;
    // the patch kernel copies input rows straight into LDS and cannot touch them on the way
    for (int i = 0; i < (q.pre_act ? 0 : kNumPatchVariants); ++i) {
        const PatchVariant &v = kPatchVariants[i];
        for (int cb = 2; cb <= cpad && cb <= 64; cb += 2) {
            if (cpad % cb != 0) continue;
            const int rc = v.reg_class(q, cb);
            if (rc < 0) continue;
            const int nstages = (q.C + cb - 1) / cb;
            for (int sk : kSplits) {
                if (sk > nstages) break;
                cand.cfg = {v.bm, v.bn, 0, v.wm, v.wn, sk, 0, 0, 1, cb};
                model_conv(q, cand.cfg, v.threads, rc, &cand.rep);
                out->push_back(cand);
            }
        }
    }
    const long Kg = (long)q.C * q.R * q.S;
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        const long stages = (Kg + v.bk - 1) / v.bk;
        if (v.threads == 512 && !split_pays(q.K, q.R * q.S, Kg)) continue;   // pays through the splitting alone
        for (int sk : kSplits) {
            if (sk > stages) break;
            // raster 1: each XCD's workgroups take neighbouring tiles, so filter rows and the input rows
            // that neighbouring pixel tiles share are fetched into one L2 instead of eight (time
            // within 1 % of raster 0 on every layer measured, a third less traffic from the fabric)
            cand.cfg = {v.bm, v.bn, v.bk, v.wm, v.wn, sk, 0, 1, 0, 0};
            if (q.has_tap && gather_tap_major_fits(q, v.bk)) cand.cfg.layout = 2;   // never slower than layout 0
            model_conv(q, cand.cfg, v.threads, 0, &cand.rep);
            out->push_back(cand);
            // the same with the leftover tiles of the last round split (wave tiles up to 64x32:
            // with larger ones the pieces measured slower than the round they save)
            if (sk == 1 && v.wm * v.wn <= 64 * 32) {
                cand.cfg.raster = 3;
                model_conv(q, cand.cfg, v.threads, 0, &cand.rep);
                out->push_back(cand);
            }
        }
    }
}

bool pick_conv(const ConvProblem &q, polydl_tile_cfg *best, polydl_model_report *best_rep, PickLimits limits)
{
    std::vector<ConvCandidate> cands;
    conv_candidates(q, &cands);
    auto tiles = [&](const ConvCandidate &c) {
        return std::ceil((double)q.K / c.cfg.bm) * std::ceil((double)q.N * q.P * q.Q / c.cfg.bn);
    };
    auto part_bytes = [&](const ConvCandidate &c) {
        return c.cfg.split_k > 1 ? tiles(c) * c.cfg.split_k * c.cfg.bm * c.cfg.bn * 4 : 0.0;
    };
    // Parts of more than 32 MiB leave the caches, and splitting that far gains less than predicted: where it
    // was predicted 1 .. 4 % faster it was 5 .. 14 % slower (116 -> 317 3x3 on 28x28, batch 17: 78 us whole, 91 in three
    // parts), where 5 % and more, faster.
    auto rank = [&](const ConvCandidate &c) { return c.rep.predicted_us * (part_bytes(c) > 32 * 1024 * 1024 ? 1.05 : 1.0); };
    // Equal predictions are candidates held by the same data floor: of those the smaller workgroup
    // tile goes first (more workgroups, so more independent loads in flight and a shorter last round).
    auto before = [&](const ConvCandidate &c, const ConvCandidate &b) {
        const double c_us = rank(c), b_us = rank(b), tie = 1e-6 * b_us;
        if (c_us < b_us - tie) return true;
        if (c_us > b_us + tie) return false;
        return c.cfg.bm * c.cfg.bn < b.cfg.bm * b.cfg.bn;
    };
    const ConvCandidate *b = nullptr;
    bool b_fits = false;       // a variant that can be launched goes before every one that cannot
    for (const ConvCandidate &c : cands) {
        if (limits.no_scratch && (c.cfg.split_k > 1 || c.cfg.raster >= 2)) continue;
        if (!limits.pointwise && c.cfg.algo == 2) continue;
        // the fp32 row-patch kernel is no match for the split products (1.1 .. 1.7 times the time of the best of
        // those on the suite); its own predictions are not comparable to theirs
        if (c.cfg.algo == 1 && split_pays(q.K, q.R * q.S, (int64_t)q.C * q.R * q.S)) continue;
        // a call that brings its own scratch memory gets the best variant that fits it.  (Held to 32 MiB, as
        // other calls once were, 2048 -> 64 channels 3x3 on 28x28, batch 32, took 635 us instead of 467, and
        // 2048 -> 128 on 56x56 3312 instead of 2860.)
        if (q.arena && c.cfg.split_k > 1 && (part_bytes(c) > q.arena->partial_bytes || tiles(c) > q.arena->ncounters)) continue;
        const bool fits = c.cfg.algo != 0 || conv_tile_in_range(q, c.cfg.bm, c.cfg.bn);
        if (b && fits != b_fits ? fits : !b || before(c, *b)) {
            b = &c;
            b_fits = fits;
        }
    }
    if (!b) return false;
    *best = b->cfg;
    *best_rep = b->rep;
    return true;
}

// every (variant, split factor, workgroup order) pick_sgemm ranks
void sgemm_candidates(const SgemmProblem &q, std::vector<polydl_tile_cfg> *out)
{
    out->clear();
    for (int i = 0; i < kNumVariants; ++i) {
        const Variant &v = kVariants[i];
        const long stages = ((long)q.K + v.bk - 1) / v.bk;
        if (v.threads == 512 && q.K < kSgemmSplitMinReduction) continue;   // pays through the splitting alone
        // long, skinny reductions (few output tiles) want many parts
        static const int kSgemmSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128};
        for (int sk : kSgemmSplits) {
            if (sk > stages) break;
            for (int raster = 0; raster < 2; ++raster)
                out->push_back(polydl_tile_cfg{v.bm, v.bn, v.bk, v.wm, v.wn, sk, 0, raster, 0, 0});
        }
    }
}

bool pick_sgemm(const SgemmProblem &q, polydl_tile_cfg *best, polydl_model_report *best_rep, bool no_scratch)
{
    bool have = false;
    int best_order = 0;
    polydl_model_report rep;
    std::vector<polydl_tile_cfg> cands;
    sgemm_candidates(q, &cands);
    for (const polydl_tile_cfg &c : cands) {
        if (no_scratch && c.split_k > 1) continue;
        model_sgemm(q, c, (c.bm / c.wm) * (c.bn / c.wn) * 64, &rep);
        if (c.raster == 1) rep.predicted_us *= 0.999;   // ties go to the XCD-aware order
        // a variant that can be launched goes before every one that cannot, and the smaller error of split
        // operands before the 128x256 tile's speed on short products (4096x4096x32: 21 us against 24.5)
        const int order = 2 * sgemm_tile_in_range(q, c.bm, c.bn, c.bk) +
                          (split_products(c.bk, c.wm, c.wn) && q.K >= kSgemmSplitMinReduction);
        if (have && order != best_order ? order > best_order : !have || rep.predicted_us < best_rep->predicted_us) {
            *best = c;
            *best_rep = rep;
            have = true;
            best_order = order;
        }
    }
    return have;
}

}  // namespace polydl
