// hawkes_loglik.hip -- O(N^2) spatiotemporal Hawkes log-likelihood and its
// gradient on gfx950 (MI355X), behind the C ABI declared in include/hawkes.h.
//
// Model: paper Section 2.1 (equations "fixed", "varying", "model" and the
// compensator after the R^2 approximation); floor of Section 2.3.1; row
// slices of Section 2.3.2.  See include/hawkes.h for the exact definition.
//
// Pipeline of one call (all on the caller's stream, no allocation):
//   1. k_stage                     tie-group ids, tile time ranges, data checks and, for
//                                  FP32, the per-theta source records in SoA layout
//   2. k_plan                      status words; the tiles each target block visits and,
//                                  for the symmetric sweep, the numbering of its cells
//                                  (1 and 2 in one launch at small n: k_stage_plan; skip
//                                  mode at larger n: k_stage_bounds, staging with lower
//                                  bounds of the rows' rates)
//   3. k_pair_f32 / k_pair_f64     the pair sweep: per target row, six sums over the
//                                  sources of one source range, in passes; k_fold adds
//                                  a pass's partial sums to the per-row accumulators
//   4. k_fold<.., true>            the last pass's fold, and per row: lambda_n, log,
//                                  gradient terms, compensator (FP64); FP32 rows whose
//                                  sums are underflow-limited go on a rescue list
//   5. k_finish_rows               those rows again, every pair in FP64, and
//                                  the fixed-order FP64 sums of all rows
//
// Pair sums of target n (u_m = s_m^-2):
//   S0 = sum_{t_m != t_n} b_nm,  Sd2 = sum b d^2,  Sdt2 = sum b dt^2,
//   G0 = sum_{t_m < t_n} u_m e_nm,  G1 = sum u_m e (u_m d^2),  G2 = sum u_m e dt,
//   b_nm = exp(-d^2/(2 tau_x^2) - dt^2/(2 tau_t^2)),  e_nm = exp(-u_m d^2/(2 h0^2) - omega dt).
// With c_b = 1/((2 pi)^1.5 tau_x^2 tau_t) and c_g = omega/(2 pi h0^2):
//   lambda_n = mu c_b S0 + xi c_g G0, and every d lambda_n / d theta is a
//   linear combination of the six sums.
//
// Work decomposition: TS = 256 sources per tile are staged through LDS
// (double buffered) and read by all lanes as broadcasts; a target block of
// TB = 512 rows sits in registers (2 per lane).  Each (target block, tile)
// pair is classified from the tile's and the block's time ranges: CAUSAL
// (every source strictly earlier than every target: background +
// triggering, no masks), ANTI (every source strictly later: background
// only) or MIXED (per-pair masks from tie-group ids).  Causality is never
// decided from rounded times.  The background kernel is symmetric in the
// pair, so over the whole event set each strictly ordered pair of blocks is
// swept once, from the later block, and its background terms are added to
// both blocks' rows (the FP32 symmetric sweep); a row range sweeps all its
// tiles.  Partial sums go to per-source-range slots that the finalize adds
// in a fixed order, so results are bitwise reproducible.
//
// Several parameter vectors (hawkes_loglik_batch): k_pair_f32_batch sweeps the
// forward sums of two vectors at once, forming each pair's differences and
// squared distance once; each vector then takes its own finalize and reduction.
//
// Skip mode (HAWKES_FP32_SKIP): the same FP32 sweep without the pairs whose
// background term is exactly zero in FP32 because the time gap alone puts its
// exponent past the subnormal range, and (large event sets) without those far
// terms that all together are below 2^-60 of the row's rate; same results,
// less work on long spans.
//
// FP32 arithmetic (precision HAWKES_FP32):
//  * positions are pre-scaled in FP64 by sqrt(log2(e)/(2 tau_x^2)) and times
//    by sqrt(log2(e)/(2 tau_t^2)); the background exponent A = d2 + dt^2 is
//    formed in FP64 from them and rounded once, so no rounded per-theta
//    constant and no rounded time difference (integer-day data have only a
//    few distinct ones) enters the background;
//  * the triggering time factor is split at the tile's last time T_k:
//    exp(-omega dt) = exp(-omega (t_n - T_k)) * exp(-omega (T_k - t_m)); the
//    source factor is folded into v_m = u_m exp(-omega (T_k - t_m)) at
//    staging and the target factor is applied in FP64 per tile;
//  * FP32 partial sums of 8 terms are folded into FP64 accumulators; the
//    column sums of the symmetric sweep are FP32 sums over a wave's 128
//    targets, folded into FP64 per tile.

#include <hip/hip_runtime.h>

#include <cfloat>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <type_traits>

#include "hawkes.h"
#include "hawkes_common.h"

namespace hawkes {

namespace {

// Compile-time shape of the FP32 sweep (defaults measured fastest on gfx950;
// the macros exist so that other shapes can be built and timed).
#ifndef HAWKES_KT
#define HAWKES_KT 2
#endif
#ifndef HAWKES_GS
#define HAWKES_GS 8
#endif

constexpr int TS = 256;                   // sources per LDS tile
constexpr int WG = 256;                   // threads per workgroup (4 wave64)
constexpr int NW = WG / 64;               // waves per workgroup
constexpr int KT = HAWKES_KT;             // target rows per lane
constexpr int TB = WG * KT;               // target rows per workgroup
constexpr int GS = HAWKES_GS;             // FP32 terms summed before folding into FP64
// row sweep: workgroups (target blocks x source chunks) a call aims for
constexpr int64_t DEFAULT_ROW_WGS = 32768;
constexpr int64_t MAX_ROW_WGS = 65536;
// Row groups of the symmetric sweep: one target block each up to PLAN_GROUPS
// blocks, above that at most PLAN_GROUPS groups of several.  (DEFAULT_SYM_GROUPS: the blocks up to which the
// default plan picks the width of column groups, and the groups whose cell the smallest workspace holds.)  A pass
// ends when its last workgroup does, and the chip idles for about a third of a
// cell's time: smaller cells (3 blocks x 6 tiles at 10^6 events) lose less there and
// write more partial sums.  At 10^6 events in the default workspace, full sweep /
// skip mode (waves; before its ranges followed the rates): 384 groups 338 / 199 ms,
// 489 groups 333 / 192, 652 groups 335 / 189, 977 groups 337 / 187.
constexpr int DEFAULT_SYM_GROUPS = 384;
constexpr int PLAN_GROUPS = 652;
constexpr int MAX_SYM_GROUPS = 1024;
constexpr int64_t PLAN_CUS = 256;  // CUs of the chip
// Partial sums of the sweep's workgroups ("cells") go to slots that a fold
// kernel adds into per-row FP64 accumulators after each pass over at most as
// many cells as the slot region holds; the default region is this large (or
// what one pass over every cell needs, if less): with the part linear in n,
// under 10^9 bytes of workspace at 10^6 events, 6144 cells a pass (rounded down to
// whole rounds of resident workgroups).  Each pass drains the chip at its end: in 3.7 GiB the
// full sweep of 10^6 events takes 323 ms instead of 333, the skip mode 130 instead of 140.
constexpr size_t DEFAULT_SLOT_BYTES = size_t(704) << 20;
constexpr int MAX_FUSED_THETA = 2;        // parameter vectors one batched sweep evaluates together
constexpr int64_t MAX_N = int64_t(1) << 30;
constexpr double LOG2E = 1.4426950408889634074;
constexpr float LN2F = 0.69314718055994530942f;
constexpr double LAMBDA_FLOOR = 1e-40;
// Padding sources (the tail of the last tile) sit far away in space and in
// time, so that every one of their terms is exactly 0 in both background forms
// (the uniform background has no spatial factor to rely on).  Their squared
// distances stay finite in FP32.
constexpr double PAD_COORD = 1e15;
constexpr double PAD_TIME = -1e15;

// Mean relative error of v_exp_f32 on gfx950, measured over 2^30 FP32
// arguments spread uniformly on [-30, 0] (and, to within 2e-10, on [-12, 0]
// and [-100, -30]): every FP32 pair term carries exactly one hardware exp2,
// so the FP32 sums are divided by (1 + this) in FP64.
constexpr double EXP2_MEAN_REL_ERR = -3.41e-9;
// Rows whose FP32 rate may have lost more than this fraction of its value to
// FP32 underflow (terms below 2^-126) are recomputed in FP64.
constexpr double RESCUE_REL = 1e-12;
// Background exponents (in units of log2) at or above this give exp2 = 0 in
// FP32 (the smallest subnormal is 2^-149); the skip mode leaves out pairs
// whose scaled time gap alone reaches it.
constexpr double SKIP_EXPONENT = 160.0;
// The skip mode also leaves out source tiles so far before a target block
// that each triggering term is below 2^-160 (u_max exp(-omega gap)): terms
// that underflow to zero in FP32 arithmetic and change no FP64 sum here.
constexpr double TRIG_SKIP_EXPONENT = 160.0;
// Nearer than that it leaves out terms which together are below 2^-60 of the row's
// rate (the gradient weighs them up to 2^7 times more): from the number and size of the terms on one
// side and a lower bound of the rate (rate_bounds) on the other.
constexpr double RATE_BITS = 60.0;
constexpr double LN2 = 0.69314718055994530942;

constexpr int STATUS_ORDER = 1;
constexpr int STATUS_DATA = 2;

enum TileClass { CAUSAL = 0, ANTI = 1, MIXED = 2 };

inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }
inline bool is_fp32(int precision) { return precision == HAWKES_FP32 || precision == HAWKES_FP32_SKIP; }
inline bool valid_precision(int precision) { return precision == HAWKES_FP64 || is_fp32(precision); }
inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------ layout

// Cells of the symmetric sweep: row groups of rr target blocks against column
// groups of cg sources (whole tiles, or a 16-source multiple that divides a
// tile), one workgroup per pair of groups it needs.
struct SymPlan {
    int rr = 1, cg = TB, num_gr = 0, num_gc = 0;
};

SymPlan finish_sym_plan(int64_t n, int rr, int cg)
{
    SymPlan S;
    S.rr = rr;
    S.cg = cg;
    S.num_gr = int(ceil_div(ceil_div(n, TB), rr));
    S.num_gc = int(ceil_div(ceil_div(n, TS) * TS, cg));
    return S;
}

// `groups` row groups and as many column groups (hawkes_options.symmetric_groups).
SymPlan make_sym_plan(int64_t n, int groups)
{
    const int rr = int(ceil_div(ceil_div(n, TB), groups));
    return finish_sym_plan(n, rr, rr * TB);
}

// The default plan.  Above 384 blocks row groups and column groups hold as many events, one block up to 652
// blocks and several from there.  Below, a row
// group is one block, and what counts is how its cells fill the chip: a cell of
// 512 sources is 512 dependent steps of its waves, and few of them leave most
// of the chip idle (at 2,000 events 16 cells took 93 us, 160 of 32 sources take
// 13).  Up to one cell per CU, as narrow as gives that many (a wider cell is
// longer, more cells than CUs are packed three to a CU while others idle); at most
// 256 sources, since from there on several rounds of narrower ones are shorter.
// Measured calls (FP32 gradient, us) for widths 32 / 64 / 128 / 256 / 512: 2,000
// events 34 / 36 / 47 / 63 / 98, 5,000 events 57 / 54 / 48 / 63 / 98, 7,000 events
// 74 / 65 / 70 / 65 / 99.  Beside the lines at 40 and 96 blocks, for 64 / 128 / 256 / 512 (skip mode, waves):
//   16,000 events  156 / 145 / 151 / 183  (120 / 115 / 115 / 184)
//   20,480 events  227 / 199 / 200 / 229  (161 / 152 / 156 / 204)
//   26,000 events  361 / 300 / 293 / 318  (222 / 198 / 200 / 212)
//   45,000 events  1080 / 872 / 754 / 767  (612 / 479 / 438 / 461)
//   49,152 events  1278 / 1023 / 901 / 900  (716 / 560 / 507 / 523)
//   60,000 events  1955 / 1538 / 1364 / 1319  (1047 / 833 / 726 / 727)
SymPlan default_sym_plan(int64_t n)
{
    const int64_t tb = ceil_div(n, TB);
    if (tb > DEFAULT_SYM_GROUPS)
        return make_sym_plan(n, PLAN_GROUPS);
    for (int cg = 32; cg <= 256; cg *= 2)
        if (tb * (tb + 1) / 2 * (TB / cg) <= PLAN_CUS)  // the triangle of block pairs
            return finish_sym_plan(n, 1, cg);
    return finish_sym_plan(n, 1, tb <= 40 ? 128 : (tb <= 96 ? 256 : TB));
}

// Per-source FP32 record fields in 8-byte slots (pairs), so that one index
// scale addresses every field of a source in LDS.
struct DeltaGroup {
    float d;  // T_k - t_m: the source's time offset from its tile's last time
    int g;    // tie-group id
};

// Workspace: a fixed part that grows linearly with n (staged records, per-row
// accumulators and values) followed by the slot region of the passes, whose
// size is whatever the caller's workspace leaves (at least one cell).
struct Layout {
    int64_t n = 0, n_pad = 0, num_tiles = 0, max_blocks = 0, rows_cap = 0;
    size_t status = 0, g = 0, tile = 0, rowvals = 0, rescue = 0;
    size_t xs = 0, ys = 0, tsd = 0, r2 = 0, v2 = 0, u2 = 0, dg = 0;
    size_t kstrict = 0, kend = 0, gchi = 0, gclo = 0, rowstart = 0;
    size_t acc = 0, blocks = 0, slots = 0, fixed = 0;
    size_t total = 0;    // the size hawkes_workspace_bytes returns
    size_t minimum = 0;  // the fixed part and one cell of the default plans
};

// Bytes of one cell's slot: row sums (6 per row) and, in the symmetric sweep,
// column sums (3 per source) of its group's events.
inline size_t sym_cell_bytes(const SymPlan &S)
{
    return sizeof(double) * (6 * size_t(S.rr) * TB + 3 * size_t(S.cg));
}
inline size_t row_cell_bytes() { return sizeof(double) * 6 * size_t(TB); }

// Work plan of the row sweep: target blocks over the row range, source chunks.
struct Plan {
    int64_t rows = 0, num_tb = 0, rows_pad = 0, chunk_tiles = 0, num_chunks = 0;
};

Plan make_plan(int64_t rows, int64_t num_tiles, int64_t target_wgs)
{
    Plan P;
    P.rows = rows;
    P.num_tb = ceil_div(rows, TB);
    P.rows_pad = P.num_tb * TB;
    int64_t want = ceil_div(target_wgs, P.num_tb);
    if (want < 1)
        want = 1;
    if (want > num_tiles)
        want = num_tiles;
    P.chunk_tiles = ceil_div(num_tiles, want);
    P.num_chunks = ceil_div(num_tiles, P.chunk_tiles);
    return P;
}

// Slot bytes a call with the default tuning needs for a single pass (the
// symmetric sweep's bound counts every row group x column group cell).
size_t single_pass_bytes(int64_t n)
{
    const SymPlan S = default_sym_plan(n);
    const size_t sym = size_t(S.num_gr) * size_t(S.num_gc) * sym_cell_bytes(S);
    const Plan P = make_plan(n, ceil_div(n, TS), DEFAULT_ROW_WGS);
    const size_t row = size_t(P.num_tb) * size_t(P.num_chunks) * row_cell_bytes();
    return sym > row ? sym : row;
}

Layout make_layout(int64_t n, int precision)
{
    Layout L;
    L.n = n;
    L.num_tiles = ceil_div(n, TS);
    L.n_pad = L.num_tiles * TS;
    const int64_t tb_max = ceil_div(n, TB);
    L.max_blocks = ceil_div(n, WG);
    L.rows_cap = tb_max * TB;

    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    L.status = take(256);
    L.g = take(sizeof(int) * L.n_pad);
    L.tile = take(sizeof(double) * 3 * L.num_tiles);
    if (is_fp32(precision)) {
        L.xs = take(sizeof(double) * L.n_pad);
        L.ys = take(sizeof(double) * L.n_pad);
        L.tsd = take(sizeof(double) * L.n_pad);
        // r_m and v_m of each vector a batched sweep evaluates (the single sweep uses the first)
        L.r2 = take(sizeof(float2) * L.n_pad * MAX_FUSED_THETA);
        L.v2 = take(sizeof(float2) * L.n_pad * MAX_FUSED_THETA);
        L.u2 = take(sizeof(float2) * L.n_pad);
        L.dg = take(sizeof(DeltaGroup) * L.n_pad);
    }
    L.kstrict = take(sizeof(int) * tb_max);
    L.kend = take(sizeof(int) * tb_max);
    L.gchi = take(sizeof(int) * MAX_SYM_GROUPS);
    L.gclo = take(sizeof(int) * MAX_SYM_GROUPS);
    L.rowstart = take(sizeof(int) * (MAX_SYM_GROUPS + 1));  // + the symmetric plan's cell count
    // per-row FP64 accumulators of the folded partial sums: 6 row sums, 3 column sums
    L.acc = take(sizeof(double) * 9 * L.rows_cap);
    L.blocks = take(sizeof(double) * 7 * L.max_blocks);  // staging results, then rescue masks
    L.rowvals = take(sizeof(double) * 7 * L.rows_cap);
    L.rescue = take(sizeof(int) * L.rows_cap);
    L.slots = off;
    L.fixed = off;
    size_t slot_bytes = single_pass_bytes(n);
    if (slot_bytes > DEFAULT_SLOT_BYTES)
        slot_bytes = DEFAULT_SLOT_BYTES;
    // at least one square cell of up to DEFAULT_SYM_GROUPS groups, which is never smaller than a cell
    // of the default plans
    const size_t one_cell = sym_cell_bytes(make_sym_plan(n, DEFAULT_SYM_GROUPS));
    if (slot_bytes < one_cell)
        slot_bytes = one_cell;
    L.total = align256(off + slot_bytes);
    L.minimum = align256(off + one_cell);
    return L;
}

// Device view of the cells of a sweep, numbered in launch order: row groups
// from the latest down, and within a row group the column groups it reaches
// from the earliest up.  Symmetric sweep: row group gr reaches column groups
// gclo[gr]..gchi[gr] (both nondecreasing in gr, from the device plan) and its
// first cell is rowstart[gr]; row sweep (rowstart == nullptr): every target
// block takes every chunk.
struct CellMap {
    const int *rowstart = nullptr, *gchi = nullptr, *gclo = nullptr;
    const int *total = nullptr;  // symmetric sweep: the plan's cell count
    int num_gr = 0, num_gc = 0;
    int cell0 = 0;               // first cell of the pass being launched
    int ncells = 0;              // cells of that pass (its workgroups)
};

// Cell of workgroup w of the current pass and its slot (false: past the last cell).  A pass's
// workgroups take its cells in reverse order: within a row group the cells nearest the diagonal,
// the costliest when far pairs are skipped, start first, and the pass ends on cheaper ones.
// Called by whole waves.
__device__ inline bool map_cell(const CellMap &m, unsigned w, int &gr, int &gc, int &slot)
{
    slot = m.ncells - 1 - int(w);
    const int c = m.cell0 + slot;
    if (!m.rowstart) {
        if (c >= m.num_gr * m.num_gc)
            return false;
        gr = m.num_gr - 1 - c / m.num_gc;
        gc = c % m.num_gc;
        return true;
    }
    // rowstart decreases with gr and rowstart[num_gr - 1] = 0: c belongs to the
    // group whose number is the count of entries above c.  The wave's lanes
    // search 64-ary (num_gr <= 1024): one round of loads up to 64 groups, else two
    const int lane = threadIdx.x & 63;
    const int stride = (m.num_gr + 63) >> 6;
    const int i0 = lane * stride < m.num_gr ? lane * stride : m.num_gr - 1;
    int start = m.rowstart[i0], first = m.gclo[i0];
    const int total = *m.total;
    const int k = __popcll(__ballot(lane * stride < m.num_gr && start > c));
    if (c >= total)
        return false;
    int from = k;  // lane holding the group's rowstart and gclo
    gr = k;
    if (stride > 1) {
        const int base = k > 0 ? (k - 1) * stride + 1 : 0;
        const int i = base + lane < m.num_gr ? base + lane : m.num_gr - 1;
        start = m.rowstart[i];
        first = m.gclo[i];
        from = __popcll(__ballot(k > 0 && lane < stride - 1 && base + lane < m.num_gr && start > c));
        gr = base + from;
    }
    gc = __builtin_amdgcn_readlane(first, from) + c - __builtin_amdgcn_readlane(start, from);
    return true;
}

// ------------------------------------------------------------- kernels

// Status words, all written by k_plan: [0] data-check flags; 8-byte word
// STATUS_UMAX the largest u_m = s_m^-2; [STATUS_RESCUE + z] the number of rows
// on the rescue list of vector z and [STATUS_TICKET + z] the workgroups of
// k_finish_rows that are done with it.
constexpr int STATUS_UMAX = 1;
constexpr int STATUS_RESCUE = 4;
constexpr int STATUS_TICKET = STATUS_RESCUE + MAX_FUSED_THETA;

__global__ void k_zero_outputs(double *loglik, double *grad)
{
    const int i = threadIdx.x;
    if (i == 0 && loglik)
        loglik[0] = 0.0;
    if (i < 6 && grad)
        grad[i] = 0.0;
}

// Splits an FP64 value into an FP32 pair hi + lo (hi = nearest FP32).
__device__ inline void split_f32(double v, float &hi, float &lo)
{
    hi = float(v);
    lo = float(v - double(hi));
}

// Per-workgroup result of the staging, gathered by k_plan.
struct StageBlock {
    double umax;
    double flags;
};

struct StageArgs {
    const double *t, *x, *y, *s;
    int64_t n, n_pad;
    int *g;
    double *tile;
    StageBlock *blocks;
    // FP32 records of the first vector, and r_m, v_m of num_theta vectors (theta_stride apart)
    double *xs, *ys, *tsd;
    float2 *r2, *v2, *u2;
    DeltaGroup *dg;
    int64_t theta_stride;
    int num_theta;
    double sx, st;
    double rr[MAX_FUSED_THETA], omega[MAX_FUSED_THETA];
};

// Lower bound of ti = t[i] in the (sorted) time array, prev = t[i - 1]: the event itself unless
// it is tied; then steps back of doubling length and a binary search in the last one.
__device__ inline int64_t first_of_ties(const double *__restrict__ t, int64_t i, double ti, double prev)
{
    if (i == 0 || prev < ti)
        return i;
    int64_t hi = i - 1, step = 1;  // t[hi] >= ti
    while (hi - step >= 0 && !(t[hi - step] < ti)) {
        hi -= step;
        step *= 2;
    }
    int64_t lo = (hi - step >= 0) ? hi - step + 1 : 0;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (t[mid] < ti)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// One pass over the events: tie-group ids (index of the first event with the
// same time), tile time ranges, the device-side data checks and the largest
// u_m; with F32 also the per-theta source records of the FP32 sweep (SoA of
// 8-byte fields, padded to whole tiles): positions and times pre-scaled in
// FP64; r_m = u_m (tau_x/h0)^2, v_m = u_m exp(-omega (T_k - t_m)) and u_m as
// FP32 hi + lo pairs, so that no rounding is shared by many pairs (all sources
// of the paper's model 1 have one u; integer-day times give few distinct
// T_k - t_m); the time offset T_k - t_m with the tie-group id.
// HBM-bound at large n (32 B read, 60 B written per event); at small n a
// launch's latency, so everything that needs one pass over the events is here.
// Event i < n_pad (padding from n on); its flags and u_m are added to the thread's.
template <bool F32>
__device__ __forceinline__ void stage_event(const StageArgs &a, int64_t i, double &umax, int &flags)
{
    double u = 0.0;
    if (i >= a.n) {
        a.g[i] = INT_MAX;
        if (F32) {
            a.xs[i] = PAD_COORD;
            a.ys[i] = PAD_COORD;
            a.tsd[i] = PAD_TIME;
            a.u2[i] = make_float2(0.0f, 0.0f);
            for (int z = 0; z < a.num_theta; ++z)
                a.r2[z * a.theta_stride + i] = a.v2[z * a.theta_stride + i] = make_float2(0.0f, 0.0f);
            a.dg[i] = DeltaGroup{0.0f, INT_MAX};
        }
    } else {
        const double ti = a.t[i], xi = a.x[i], yi = a.y[i], si = a.s[i];
        const int64_t k = i / TS;
        const double tlast = a.t[((k + 1) * TS < a.n ? (k + 1) * TS : a.n) - 1];
        const double prev = (i > 0) ? a.t[i - 1] : ti;
        const double next = (i + 1 < a.n) ? a.t[i + 1] : ti;
        u = 1.0 / (si * si);
        if (!isfinite(ti) || !isfinite(xi) || !isfinite(yi) || !isfinite(si) || !(si > 0.0))
            flags |= STATUS_DATA;
        if (next < ti)
            flags |= STATUS_ORDER;
        const int64_t lo = first_of_ties(a.t, i, ti, prev);
        a.g[i] = int(lo);
        if (i % TS == 0) {
            a.tile[3 * k + 0] = ti;
            a.tile[3 * k + 1] = tlast;
        }
        if (F32) {
            const double d = tlast - ti;
            a.xs[i] = xi * a.sx;
            a.ys[i] = yi * a.sx;
            a.tsd[i] = ti * a.st;
            float hi, lo32;
            for (int z = 0; z < a.num_theta; ++z) {
                split_f32(u * a.rr[z], hi, lo32);
                a.r2[z * a.theta_stride + i] = make_float2(hi, lo32);
                split_f32(u * exp(-a.omega[z] * d), hi, lo32);
                a.v2[z * a.theta_stride + i] = make_float2(hi, lo32);
            }
            split_f32(u, hi, lo32);
            a.u2[i] = make_float2(hi, lo32);
            a.dg[i] = DeltaGroup{float(d), int(lo)};
        }
    }
    umax = fmax(umax, (isfinite(u) && u > 0.0) ? u : 0.0);  // bad values are flagged above
}

// Workgroup-wide largest u_m and union of the flags, in every thread (WAVES waves).
template <int WAVES>
__device__ __forceinline__ void join_stage(double &u, int &flags)
{
    __shared__ double red_u[WAVES];
    __shared__ int red_f[WAVES];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        u = fmax(u, __shfl_xor(u, o));
        flags |= __shfl_xor(flags, o);
    }
    if ((threadIdx.x & 63) == 0) {
        red_u[threadIdx.x >> 6] = u;
        red_f[threadIdx.x >> 6] = flags;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        u = fmax(u, red_u[w]);
        flags |= red_f[w];
    }
}

template <bool F32>
__global__ __launch_bounds__(256) void k_stage(StageArgs a)
{
    double u = 0.0;
    int flags = 0;
    stage_event<F32>(a, int64_t(blockIdx.x) * 256 + threadIdx.x, u, flags);
    join_stage<4>(u, flags);
    if (threadIdx.x == 0)
        a.blocks[blockIdx.x] = StageBlock{u, double(flags)};
}

// Lower bounds of the rates of BOUND_ROWS rows (skip mode): over them and over the call's vectors,
// the least log2 of lambda against the largest background and triggering term an event can add
// (c_b max(mu, 1) and c_g u exp(..) max(xi, 1): also what bounds the gradient in mu and xi), and the
// sum of the rows' own u.
//   lambda_n is at least its largest single term; here that of the `sources` events before the
// rows (before their ties), with the rows' last time in place of their own.  Differences in FP64,
// exponents in FP32: their rounding is some 1e-5 of a bit.
//   Taken above BOUND_EVENTS events: it costs 10-15 us of small launches at such sizes and takes 20-25%
// off the pair sweep (12,000 events over 1000 days 84 us without, 85 with; 16,000 113, 113; 20,000
// 150, 144; 100,000 over 1200 days 1985, 1646; 1e6 184, 139 ms).  Its VALU work, some 12
// instructions per row and event, hides behind nothing: 0.3 ms per 512 events at 1e6 rows.
constexpr int64_t BOUND_EVENTS = 16384;
constexpr int BOUND_ROWS = 64;
constexpr int BOUND_SOURCES = 512;        // staged at a time
constexpr int64_t MAX_BOUND_SOURCES = 4096;
constexpr int BOUND_WAVES = 16;
struct RateBound {
    float bg, trig, usum;
};
struct BoundArgs {
    const double *t, *x, *y, *s;
    int64_t n;
    RateBound *out;
    int groups;       // of BOUND_ROWS rows
    int sources;      // whole multiples of BOUND_SOURCES
    double min_span;  // shorter event sets have no pair far enough apart: no bounds
    float ax[MAX_FUSED_THETA], at[MAX_FUSED_THETA], qh[MAX_FUSED_THETA], w[MAX_FUSED_THETA];
    // log2 of mu c_b, xi c_g, c_b max(mu, 1), c_g max(xi, 1)
    float bg[MAX_FUSED_THETA], trig[MAX_FUSED_THETA], bg_unit[MAX_FUSED_THETA], trig_unit[MAX_FUSED_THETA];
};
template <int NT>
__device__ void rate_bounds(const BoundArgs &a, int group)
{
    static_assert(BOUND_ROWS == 64 && BOUND_SOURCES <= 64 * BOUND_WAVES, "a lane per row, a thread per source");
    static_assert(BOUND_SOURCES % BOUND_WAVES == 0, "whole shares");
    __shared__ double2 lxy[BOUND_SOURCES];
    __shared__ float lu[BOUND_SOURCES];
    __shared__ float2 lbg[NT][BOUND_SOURCES];
    __shared__ float best[NT][BOUND_WAVES][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (!(a.t[a.n - 1] - a.t[0] > a.min_span))
        return;
    const int64_t r0 = int64_t(group) * BOUND_ROWS;
    const int64_t last = r0 + BOUND_ROWS < a.n ? r0 + BOUND_ROWS - 1 : a.n - 1;
    const int64_t i = r0 + lane < a.n ? r0 + lane : a.n - 1;
    const double xn = a.x[i], yn = a.y[i], sn = a.s[i];
    const double t_first = a.t[r0], t_last = a.t[last], prev = r0 > 0 ? a.t[r0 - 1] : t_first;
    const int64_t end = first_of_ties(a.t, r0, t_first, prev);
    float A[NT], G[NT];
#pragma unroll
    for (int z = 0; z < NT; ++z) {
        A[z] = HUGE_VALF;
        G[z] = -HUGE_VALF;
    }
    for (int64_t m0 = end - BOUND_SOURCES; m0 > end - a.sources - BOUND_SOURCES && m0 > -BOUND_SOURCES;
         m0 -= BOUND_SOURCES) {
        if (tid < BOUND_SOURCES) {
            const int64_t m = m0 + tid;
            const bool in = m >= 0;
            const int64_t mc = in ? m : 0;
            const double sm = a.s[mc];
            const float u = float(1.0 / (sm * sm)), dt = float(t_last - a.t[mc]);
            lxy[tid] = {a.x[mc], a.y[mc]};
            lu[tid] = u;
#pragma unroll
            for (int z = 0; z < NT; ++z)
                lbg[z][tid] = in ? make_float2(a.at[z] * dt * dt, log2f(u) - a.w[z] * dt)
                                 : make_float2(HUGE_VALF, -HUGE_VALF);
        }
        __syncthreads();
        constexpr int SHARE = BOUND_SOURCES / BOUND_WAVES;
#pragma unroll 8
        for (int j = wave * SHARE; j < (wave + 1) * SHARE; ++j) {
            const float dx = float(xn - lxy[j].x), dy = float(yn - lxy[j].y);
            const float d2 = fmaf(dx, dx, dy * dy), u = lu[j];
#pragma unroll
            for (int z = 0; z < NT; ++z) {
                A[z] = fminf(A[z], fmaf(a.ax[z], d2, lbg[z][j].x));
                G[z] = fmaxf(G[z], fmaf(-a.qh[z] * u, d2, lbg[z][j].y));
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int z = 0; z < NT; ++z)
        best[z][wave][lane] = fmaxf(a.bg[z] - A[z], a.trig[z] + G[z]);
    __syncthreads();
    if (wave > 0)
        return;
    RateBound v = {HUGE_VALF, HUGE_VALF, r0 + lane < a.n ? fmaxf(float(1.0 / (sn * sn)), FLT_MIN) : 0.0f};
#pragma unroll
    for (int z = 0; z < NT; ++z) {
        float rate = best[z][0][lane];
#pragma unroll
        for (int k = 1; k < BOUND_WAVES; ++k)
            rate = fmaxf(rate, best[z][k][lane]);
        v.bg = fminf(v.bg, rate - a.bg_unit[z]);
        v.trig = fminf(v.trig, rate - a.trig_unit[z]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        v.bg = fminf(v.bg, __shfl_xor(v.bg, o));
        v.trig = fminf(v.trig, __shfl_xor(v.trig, o));
        v.usum += __shfl_xor(v.usum, o);
    }
    if (lane == 0)
        a.out[group] = v;
}

// Skip mode: staging and the rows' bounds in one launch, the bounds' workgroups first (both take
// a few dependent loads at small n).
template <int NT>
__global__ __launch_bounds__(64 * BOUND_WAVES) void k_stage_bounds(StageArgs s, BoundArgs b)
{
    if (int(blockIdx.x) < b.groups) {
        rate_bounds<NT>(b, blockIdx.x);
        return;
    }
    const int64_t block = int64_t(blockIdx.x) - b.groups, i = block * (64 * BOUND_WAVES) + threadIdx.x;
    double u = 0.0;
    int flags = 0;
    if (i < s.n_pad)
        stage_event<true>(s, i, u, flags);
    join_stage<BOUND_WAVES>(u, flags);
    if (threadIdx.x == 0)
        s.blocks[block] = StageBlock{u, double(flags)};
}

struct PairF32 {
    const double *xs, *ys, *tsd, *t;
    const float2 *r2, *v2, *u2;  // (hi, lo) of r_m, v_m, u_m
    const DeltaGroup *dg;
    const int *g;
    const double *tile;
    const int *kstrict, *kend;  // tile bounds of each target block (k_plan)
    CellMap cells;  // the cells of the sweep and the first one of this pass
    double *srow;   // [slot][6][ge]: a cell's row sums of its row group's rows (2 planes without the gradient)
    double *scol;   // [slot][3][cg]: its column group's background column sums (1 plane without the gradient)
    int ge;         // rows per row group (slot stride)
    int row_begin, row_end, rows_pad, num_tiles, num_tb;  // indices below 2^31 (n <= 2^30)
    int rr, cg;     // target blocks per row group, sources per column group
    int sym;
    // Skip mode: tiles further before a block than the gaps of the block and of
    // their own events (TileWord) sweep the triggering terms only; tiles before
    // the block's first one are not visited.
    int trig_cull;
    double omega, inv_st, out_s1, out_s2, out_g1, out_exp;
    double w2;  // omega * log2(e) / time scale: the triggering exponent per scaled day
};

// Days before a target from which on every triggering term is below u_max
// exp(-omega gap) < 2^-TRIG_SKIP_EXPONENT; no smaller than skip_gap, so that the
// background terms there are exactly zero too.
__device__ inline double trig_cull_gap(double umax, double omega, double skip_gap)
{
    const double tg = (log(umax) + TRIG_SKIP_EXPONENT * LN2) / omega;
    return (tg > skip_gap) ? tg : skip_gap;
}

// First tile whose last time is within gap days of a block that starts at t_lo.
__device__ inline int first_tile_within(const double *__restrict__ tile, int num_tiles, double t_lo, double gap)
{
    const double limit = t_lo - gap;
    int lo = 0, hi = num_tiles;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tile[3 * mid + 1] < limit)
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// First tile whose first time is more than gap days after a block that ends at t_hi.
__device__ inline int first_tile_after(const double *__restrict__ tile, int num_tiles, double t_hi, double gap)
{
    const double limit = t_hi + gap;
    int lo = 0, hi = num_tiles;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (tile[3 * mid + 0] > limit)
            hi = mid;
        else
            lo = mid + 1;
    }
    return lo;
}

// Third word of a tile's record (first time, last time, word): with trig_cull that of
// tile KT b holds block b's first tile and the days from which on a background term
// is left out of its rows' sums.
struct TileWord {
    int klo;
    float gap;
    __device__ int gap_bits() const { return __float_as_int(gap); }
};
__device__ inline TileWord tile_word(const double *__restrict__ tile, int k)
{
    return *reinterpret_cast<const TileWord *>(tile + 3 * k + 2);
}

// Pair geometry: the scaled squared distance D and the background exponent
// A = D + dt'^2, differences and squares in FP64, D and A each rounded once
// to FP32.
__device__ inline void geom_da(double xn, double yn, double tn, double xm, double ym, double tm, float &D, float &A)
{
    const double dx = xn - xm, dy = yn - ym, dt = tn - tm;
    const double d2 = fma(dy, dy, dx * dx);
    D = float(d2);
    A = float(fma(dt, dt, d2));
}
__device__ inline float geom_d(double xn, double yn, double xm, double ym)
{
    const double dx = xn - xm, dy = yn - ym;
    return float(fma(dy, dy, dx * dx));
}
// Spatially uniform background: the exponent is the scaled time gap alone,
// A = dt'^2, so with tied times (integer days) many pairs share one value of
// A and its FP32 rounding would not average out; A is split into a hi part
// (the exp2 argument) and a lo part that corrects the term to first order.
__device__ inline void geom_da_uni(double xn, double yn, double tn, double xm, double ym, double tm, float &D,
                                   float &A, float &Alo)
{
    const double dx = xn - xm, dy = yn - ym, dt = tn - tm;
    D = float(fma(dy, dy, dx * dx));
    const double a2 = dt * dt;
    A = float(a2);
    Alo = float(a2 - double(A));
}

// Column sums of the symmetric sweep.  Within each row of 16 lanes, the
// lanes take the 16 sources of a subgroup in rotation: at step j lane i takes
// source (i + j) mod 16, and the FP32 column accumulators of a source move
// with it (row_ror:15: lane i reads lane (i + 1) mod 16 of its row).  After 8
// steps each lane's accumulator (the row's sum over 8 steps of 2 targets) is
// put aside and a new one starts; after 16 steps the first half's sum of a
// source sits 8 lanes away from the second half's (row_ror:8) and the halves
// meet in FP64.  The four rows take the same sources at the same lane
// positions and are added by the gfx950 row swaps (below).
constexpr int DPP_ROW_ROR1 = 0x121, DPP_ROW_ROR2 = 0x122, DPP_ROW_ROR4 = 0x124, DPP_ROW_ROR8 = 0x128,
              DPP_ROW_ROR15 = 0x12F;
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v)
{
    return __builtin_amdgcn_mov_dpp(v, CTRL, 0xf, 0xf, true);
}
__device__ __forceinline__ float row_rotate_f32(float v)
{
    return __int_as_float(dpp_mov<DPP_ROW_ROR15>(__float_as_int(v)));
}
__device__ __forceinline__ double make_f64(unsigned lo, unsigned hi)
{
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
// first-half sum h (8 lanes back) plus second-half sum e of the lane's source
__device__ __forceinline__ double join_halves(float h, float e)
{
    return double(__int_as_float(dpp_mov<DPP_ROW_ROR8>(__float_as_int(h)))) + double(e);
}
// Sums over the rows of 16 lanes, rows r and r + 1 (r even) of a and of b: rows 0 and 2 of
// the result hold a's, rows 1 and 3 b's.  One swap moves a's odd rows against b's even
// rows, so that one addition serves both.
__device__ __forceinline__ double add_row_pairs(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    auto lo = __builtin_amdgcn_permlane16_swap(unsigned(ua), unsigned(ub), false, false);
    auto hi = __builtin_amdgcn_permlane16_swap(unsigned(ua >> 32), unsigned(ub >> 32), false, false);
    return make_f64(lo[0], hi[0]) + make_f64(lo[1], hi[1]);
}
// The same for the wave's halves: lanes 0-31 of the result hold a's sum, lanes 32-63 b's.
__device__ __forceinline__ double add_halves(double a, double b)
{
    const unsigned long long ua = (unsigned long long)__double_as_longlong(a);
    const unsigned long long ub = (unsigned long long)__double_as_longlong(b);
    auto lo = __builtin_amdgcn_permlane32_swap(unsigned(ua), unsigned(ub), false, false);
    auto hi = __builtin_amdgcn_permlane32_swap(unsigned(ua >> 32), unsigned(ub >> 32), false, false);
    return make_f64(lo[0], hi[0]) + make_f64(lo[1], hi[1]);
}
// Sums over the four rows of up to four values: row k of the result holds value k's,
// (row 0 + row 1) + (row 2 + row 3).  11 instructions for three values, against 30 when
// each value is summed across the rows by itself.
__device__ __forceinline__ double sum_rows4(double v0, double v1, double v2, double v3)
{
    return add_halves(add_row_pairs(v0, v1), add_row_pairs(v2, v3));
}
__device__ __forceinline__ double sum_rows2(double v0, double v1)
{
    const double s = add_row_pairs(v0, v1);
    return add_halves(s, s);
}
__device__ __forceinline__ double sum_rows_f64(double v) { return sum_rows2(v, v); }
static_assert(GS == 8, "the column rotation keeps one FP64 partial per 8-source group");

// Direct global-to-LDS load of one dword per lane (global_load_lds_dword):
// lane l's dword lands at LDS address `wave_base` + 4 l; `wave_base` must be
// the same for the whole wave.  stage_wait() waits for this wave's
// outstanding vector memory operations (vmcnt 0), which include these loads.
typedef __attribute__((address_space(1))) void global_void;
typedef __attribute__((address_space(3))) void lds_void;
__device__ __forceinline__ void lds_dma4(const void *src, void *wave_base)
{
    __builtin_amdgcn_global_load_lds((global_void *)src, (lds_void *)wave_base, 4, 0, 0);
}
__device__ __forceinline__ void stage_wait() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0)

// Rotation offsets of a lane within a 16-source subgroup of 8-byte fields: at step
// j < 8 it takes source (li + j) mod 16, at step 8 + j the one 64 bytes away
// (modulo the subgroup's 128).  A table of eight registers and one exclusive-or-
// and-add per step, against three integer instructions when formed at each step.
struct Rotation {
    int off[GS];
    __device__ __forceinline__ explicit Rotation(int li)
    {
#pragma unroll
        for (int j = 0; j < GS; ++j)
            off[j] = ((li + j) & 15) * 8;
    }
    // byte offset of step (half, j) with the subgroup's own offset base
    __device__ __forceinline__ int at(int j, int half64, int base) const { return (off[j] ^ half64) + base; }
};

// End of a source step: the sums v are up to date here, and nothing moves across.
// An unrolled source loop would otherwise hold many sources, or their not yet
// added terms, in registers and lose a wave per SIMD.
template <typename T, int N>
__device__ __forceinline__ void pin(T (&v)[N])
{
#pragma unroll
    for (int i = 0; i < N; ++i)
        asm volatile("" : "+v"(v[i]));
}
__device__ __forceinline__ void step_end()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// The FP32 fused sweep.  GRAD = false keeps only S0 and G0 (log-likelihood).
//
// Per pair (positions and times pre-scaled so that the background exponent
// is A = |x_n - x_m|^2 + (t_n - t_m)^2):
//   d2 = |x_n - x_m|^2 and A = d2 + dt^2 in FP64, each rounded once to FP32;
//   background b = exp2(-A); triggering (earlier sources) p = v_m exp2(-t1)
//   with t1 = r_m D.  Every FP32 value that many pairs would share is split
//   hi + lo, and every rounding left is of a value that varies from pair to
//   pair, so rounding errors average out instead of adding up.
//
// A workgroup owns a rectangle: the rr target blocks of row group gr (2 rows
// per lane each, one block at a time) against the cg sources of column group
// gc (whole tiles, or at small n a part of one tile).  Row sums stay in registers for a block's sweep over the
// rectangle's tiles and go to the row partials of column group gc.
//
// Symmetric sweep (whole event set).  The background term is symmetric in
// the pair, so a block pair whose times are strictly ordered is swept once,
// from the later block: each term b_nm goes to the row sums of n and, as a
// column sum, to the row sums of m.  The later block's view is then never
// swept from the earlier block.  Block pairs whose time ranges touch are
// swept from both sides, with per-tile classes as in the row sweep.  A
// wave's column sums of a tile come from the 16-lane rotation above (FP32
// over 8 steps, then FP64, then over the 4 rows); the tile's owner lanes add
// the 4 waves' sums in FP64 and add them to this row group's column partials,
// which the workgroup alone writes (so every sum keeps a fixed order and
// results are bitwise reproducible).
//
// Row sweep (a row range): every tile is swept for every block (rr = 1,
// no columns).
//
// Bound: VALU issue.  A step of the column loop (one source, two targets, their
// mirror terms) issues 48.9 VALU instructions with its share of the FP64 folds,
// column reduction and addressing, 58.7 before the steps were pinned one by one
// (zeroed sums of each group, three instructions per rotated address, a
// cross-row reduction per plane): 397 -> 338 ms at 10^6 events with the
// gradient, 2833 -> 2490 us without it at 10^5.
//
// Waves per SIMD the register budget must allow (512 registers per lane and
// SIMD): 3 with the gradient, which is also its LDS limit, 4 without (2833 ->
// 2538 us at 3 waves and 2490 at 4).
#ifndef HAWKES_WAVES_GRAD
#define HAWKES_WAVES_GRAD 3
#endif
#ifndef HAWKES_WAVES_FWD
#define HAWKES_WAVES_FWD 4
#endif
#define HK_WAVES(n) __attribute__((amdgpu_waves_per_eu(n)))
template <bool GRAD, bool UNI>
__global__ __launch_bounds__(WG) HK_WAVES(GRAD ? HAWKES_WAVES_GRAD : HAWKES_WAVES_FWD) void k_pair_f32(PairF32 a)
{
    // one tile of source records; the fields sit at fixed offsets from each
    // other, so a source's loads share one address and immediate offsets
    struct alignas(16) TileRecs {
        double x[TS], y[TS], t[TS];
        float2 r[TS], v[TS], u[TS];
        DeltaGroup dg[TS];
    };
    __shared__ TileRecs lt2[2];
    // per-wave column sums of the tile being swept (the forward sweep has one plane, and
    // with it four workgroups per CU instead of three)
    constexpr int CP = GRAD ? 3 : 1;
    __shared__ float lcol[2][CP][NW][TS];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15;
    int gr, gc, slot;
    if (!map_cell(a.cells, blockIdx.x, gr, gc, slot))
        return;
    const int b_first = gr * a.rr;
    const int b_stop = (b_first + a.rr < a.num_tb) ? b_first + a.rr : a.num_tb;
    // sources [jb, js) of the column group: tiles [kg0, kg1), of each the sources [mlo, mhi)
    const int jb = gc * a.cg, js = (jb + a.cg < a.num_tiles * TS) ? jb + a.cg : a.num_tiles * TS;
    const int kg0 = jb / TS, kg1 = (js + TS - 1) / TS;
    const int mlo = jb & (TS - 1), mhi = (a.cg < TS) ? mlo + a.cg : TS;
    const bool own = tid >= mlo && tid < mhi;  // this lane's source of a tile is in the group
    // this workgroup's slot: row sums of rows b_first * TB.., column sums of sources jb..
    const int64_t stride = a.ge;
    const int rb0 = b_first * TB;
    const int64_t cstride = a.cg;
    double *pc = a.scol + int64_t(slot) * CP * cstride;
    if (a.sym && own) {
        for (int k = kg0; k < kg1; ++k) {
            const int j = k * TS + tid - jb;
            pc[j] = 0.0;
            if (GRAD) {
                pc[cstride + j] = 0.0;
                pc[2 * cstride + j] = 0.0;
            }
        }
    }

    // Staging of tile k into LDS buffer buf by direct global-to-LDS loads: each
    // lane moves two dwords of every 8-byte-field array, landing at the wave's
    // base + 4 * lane.  The loads of the next tile run during the sweep;
    // stage_wait() (this wave's loads done) comes before the barrier that
    // publishes the tile.
    auto stage = [&](int k, int buf) {
        TileRecs &T = lt2[buf];
        // per-lane offset kept opaque, so that the compiler forms each address
        // from the array's tile base (scalar) and this offset rather than
        // holding a per-lane pointer for every array across the loop
        int o = tid;
        asm volatile("" : "+v"(o));
        const int wb = tid & ~63;
        const unsigned *xs = reinterpret_cast<const unsigned *>(a.xs + k * TS);
        const unsigned *ys = reinterpret_cast<const unsigned *>(a.ys + k * TS);
        const unsigned *ts = reinterpret_cast<const unsigned *>(a.tsd + k * TS);
        lds_dma4(xs + o, reinterpret_cast<unsigned *>(T.x) + wb);
        lds_dma4(xs + TS + o, reinterpret_cast<unsigned *>(T.x) + TS + wb);
        lds_dma4(ys + o, reinterpret_cast<unsigned *>(T.y) + wb);
        lds_dma4(ys + TS + o, reinterpret_cast<unsigned *>(T.y) + TS + wb);
        lds_dma4(ts + o, reinterpret_cast<unsigned *>(T.t) + wb);
        lds_dma4(ts + TS + o, reinterpret_cast<unsigned *>(T.t) + TS + wb);
        const unsigned *r2 = reinterpret_cast<const unsigned *>(a.r2 + k * TS);
        const unsigned *v2 = reinterpret_cast<const unsigned *>(a.v2 + k * TS);
        const unsigned *u2 = reinterpret_cast<const unsigned *>(a.u2 + k * TS);
        const unsigned *dg = reinterpret_cast<const unsigned *>(a.dg + k * TS);
        lds_dma4(r2 + o, reinterpret_cast<unsigned *>(T.r) + wb);
        lds_dma4(r2 + TS + o, reinterpret_cast<unsigned *>(T.r) + TS + wb);
        lds_dma4(v2 + o, reinterpret_cast<unsigned *>(T.v) + wb);
        lds_dma4(v2 + TS + o, reinterpret_cast<unsigned *>(T.v) + TS + wb);
        lds_dma4(u2 + o, reinterpret_cast<unsigned *>(T.u) + wb);
        lds_dma4(u2 + TS + o, reinterpret_cast<unsigned *>(T.u) + TS + wb);
        lds_dma4(dg + o, reinterpret_cast<unsigned *>(T.dg) + wb);
        lds_dma4(dg + TS + o, reinterpret_cast<unsigned *>(T.dg) + TS + wb);
    };

    const Rotation rot(li);

    for (int b = b_first; b < b_stop; ++b) {
        const int i0 = a.row_begin + b * TB;
        const int iend = (i0 + TB < a.row_end) ? i0 + TB : a.row_end;
        int k0 = kg0;
        int skip_gap = INT_MAX;  // gaps as the bits of a float >= 0, ordered like it, in scalar registers
        // the gap that the sums of tile k's own events ask for (symmetric sweep: they take column sums)
        auto tile_gap = [&](int k) { return a.sym ? tile_word(a.tile, k & ~(KT - 1)).gap_bits() : 0; };
        if (a.trig_cull) {
            const TileWord w = tile_word(a.tile, KT * b);
            skip_gap = w.gap_bits();
            k0 = (kg0 > w.klo) ? kg0 : w.klo;
            k0 = (k0 < a.num_tiles) ? k0 : a.num_tiles - 1;
        } else {
            stage(k0, 0);  // runs while the block's bounds and targets are loaded
        }
        const double t_lo = a.t[i0], t_hi = a.t[iend - 1];

        // lanes past the block's end take a target far away in space and time:
        // every one of its terms is exactly 0, so its column terms add nothing
        double xn[KT], yn[KT], tsn[KT], trn[KT];
        int gn[KT];
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            const bool in = i < iend;
            xn[q] = in ? a.xs[i] : PAD_COORD;
            yn[q] = in ? a.ys[i] : PAD_COORD;
            tsn[q] = in ? a.tsd[i] : PAD_TIME;
            trn[q] = a.t[in ? i : iend - 1];
            gn[q] = in ? a.g[i] : INT_MAX;
        }
        double acc[KT][6];
#pragma unroll
        for (int q = 0; q < KT; ++q)
#pragma unroll
            for (int z = 0; z < 6; ++z)
                acc[q][z] = 0.0;

        // tiles [0, k_strict): strictly earlier blocks, swept with column sums;
        // tiles before k_lo and from k_end on: not visited
        const int k_strict = a.kstrict[b], k_end = a.kend[b];
        const int k1 = (kg1 < k_end) ? kg1 : k_end;
        if (a.trig_cull && k0 < k1)
            stage(k0, 0);
        stage_wait();
        __syncthreads();

        double next_first = a.tile[3 * k0 + 0], next_last = a.tile[3 * k0 + 1];
        int next_gap = a.trig_cull ? tile_gap(k0) : 0;
        for (int k = k0; k < k1; ++k) {
            const int buf = (k - k0) & 1;
            const double first = next_first, last = next_last;
            const int gap = skip_gap > next_gap ? skip_gap : next_gap;
            if (k + 1 < k1) {
                stage(k + 1, buf ^ 1);  // into the buffer every wave finished reading
                next_first = a.tile[3 * k + 3];
                next_last = a.tile[3 * k + 4];
                if (a.trig_cull)
                    next_gap = tile_gap(k + 1);
            }

            const int cls = (last < t_lo) ? CAUSAL : ((first > t_hi) ? ANTI : MIXED);
            const bool trig_only = (cls == CAUSAL) && a.trig_cull && (t_lo - last > double(__int_as_float(gap)));
            const bool cols = (k < k_strict) && !trig_only;  // strictly earlier block (so CAUSAL)

            // Terms are summed in FP32 over groups of GS = 8 sources and each
            // group sum is folded into FP64.  Long FP32 running sums would round
            // away every Gaussian-tail term below half an ulp of the sum, a
            // systematic loss of ~1e-8 relative; groups of 8 keep it near 3e-10
            // and equal across the six sums (the gradient combines them with
            // heavy cancellation, so their errors must match).  Background sums go
            // straight into the accumulators; the CAUSAL triggering sums keep FP64
            // tile partials that take the target's time factor at the tile end.
            double gt[KT][3];
#pragma unroll
            for (int q = 0; q < KT; ++q)
                gt[q][0] = gt[q][1] = gt[q][2] = 0.0;

            const TileRecs &T = lt2[buf];

            if (cls != MIXED) {
                const bool causal = (cls == CAUSAL);
                // column sums (CAUSAL with columns): FP32 over 8 rotation steps, then FP64.
                // FP32 sums start at -0, the exact additive identity (x + -0 = x for every
                // x, +0 included), so the compiler can drop a sum's first addition and turn
                // fma(a, b, -0) into a product; a +0 start would cost an instruction
                const char *lbase = reinterpret_cast<const char *>(&lt2[0]);
                const int tbase = buf * int(sizeof(TileRecs));
                struct Src {
                    double x, y, t;
                    float2 r, v;
                    float d;
                };
                float f[KT][6];
                auto start_group = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < 6; ++z)
                            f[q][z] = -0.0f;
                };
                auto fold_back = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        acc[q][0] += double(f[q][0]);
                        if (GRAD) {
                            acc[q][1] += double(f[q][1]);
                            acc[q][2] += double(f[q][2]);
                        }
                    }
                };
                auto fold_trig = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        gt[q][0] += double(f[q][3]);
                        if (GRAD) {
                            gt[q][1] += double(f[q][4]);
                            gt[q][2] += double(f[q][5]);
                        }
                    }
                };
                // background + triggering terms of one source for the lane's targets;
                // adds the background terms' sums over those targets (b, b D, b A) to c0..c2
                auto causal_pair = [&](const Src &m, float &c0, float &c1, float &c2) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float D, A, Alo = 0.0f;
                        if (UNI)
                            geom_da_uni(xn[q], yn[q], tsn[q], m.x, m.y, m.t, D, A, Alo);
                        else
                            geom_da(xn[q], yn[q], tsn[q], m.x, m.y, m.t, D, A);
                        float b = __builtin_amdgcn_exp2f(-A);
                        if (UNI)
                            b = fmaf(-LN2F * Alo, b, b);
                        const float t1 = fmaf(m.r.y, D, m.r.x * D);
                        const float E = __builtin_amdgcn_exp2f(-t1);
                        const float p = fmaf(m.v.y, E, m.v.x * E);
                        f[q][0] += b;
                        f[q][3] += p;
                        c0 += b;
                        if (GRAD) {
                            if (!UNI) {
                                f[q][1] = fmaf(b, D, f[q][1]);
                                c1 = fmaf(b, D, c1);
                            }
                            f[q][2] = fmaf(b, A, f[q][2]);
                            c2 = fmaf(b, A, c2);
                            f[q][4] = fmaf(p, t1, f[q][4]);
                            f[q][5] = fmaf(p, m.d, f[q][5]);
                        }
                    }
                };
                // triggering terms only (the background terms are exactly zero)
                auto trig_pair = [&](const Src &m) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        const float D = geom_d(xn[q], yn[q], m.x, m.y);
                        const float t1 = fmaf(m.r.y, D, m.r.x * D);
                        const float E = __builtin_amdgcn_exp2f(-t1);
                        const float p = fmaf(m.v.y, E, m.v.x * E);
                        f[q][3] += p;
                        if (GRAD) {
                            f[q][4] = fmaf(p, t1, f[q][4]);
                            f[q][5] = fmaf(p, m.d, f[q][5]);
                        }
                    }
                };
                auto anti_pair = [&](const Src &m) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float D, A, Alo = 0.0f;
                        if (UNI)
                            geom_da_uni(xn[q], yn[q], tsn[q], m.x, m.y, m.t, D, A, Alo);
                        else
                            geom_da(xn[q], yn[q], tsn[q], m.x, m.y, m.t, D, A);
                        float b = __builtin_amdgcn_exp2f(-A);
                        if (UNI)
                            b = fmaf(-LN2F * Alo, b, b);
                        f[q][0] += b;
                        if (GRAD) {
                            if (!UNI)
                                f[q][1] = fmaf(b, D, f[q][1]);
                            f[q][2] = fmaf(b, A, f[q][2]);
                        }
                    }
                };
                // a group of 8 sources in order, the same for every lane: two at a time, in 16-byte
                // LDS reads whose offsets are immediates
                auto in_order = [&](int m0, auto &&pair) {
                    const char *g0 = lbase + (tbase + m0 * 8);
                    start_group();
#pragma unroll
                    for (int j = 0; j < GS; j += 2) {
                        auto two = [&](size_t field) {
                            return *reinterpret_cast<const float4 *>(g0 + field + j * 8);
                        };
                        auto twod = [&](size_t field) {
                            return *reinterpret_cast<const double2 *>(g0 + field + j * 8);
                        };
                        const double2 x = twod(offsetof(TileRecs, x)), y = twod(offsetof(TileRecs, y)),
                                      t = twod(offsetof(TileRecs, t));
                        const float4 r = two(offsetof(TileRecs, r)), v = two(offsetof(TileRecs, v)),
                                     d = two(offsetof(TileRecs, dg));
                        pair(Src{x.x, y.x, t.x, make_float2(r.x, r.y), make_float2(v.x, v.y), d.x});
                        pair(Src{x.y, y.y, t.y, make_float2(r.z, r.w), make_float2(v.z, v.w), d.z});
#pragma unroll
                        for (int q = 0; q < KT; ++q)
                            pin(f[q]);
                        step_end();
                    }
                };
                // 8 steps (half HALF) of the 16-source rotation (row sums as in the plain causal
                // loop): lane i takes source sub + ((i + 8 HALF + j) mod 16) at step j; the
                // column sums of the lane's source go to e0..e2
                auto rotate = [&](int sub, auto half, float &e0, float &e1, float &e2) {
                    constexpr int HALF = decltype(half)::value;
                    const int base = tbase + sub * 8;
                    auto take = [&](int j) {
                        const char *p = lbase + rot.at(j, 64 * HALF, base);
                        Src m;
                        m.x = *reinterpret_cast<const double *>(p + offsetof(TileRecs, x));
                        m.y = *reinterpret_cast<const double *>(p + offsetof(TileRecs, y));
                        m.t = *reinterpret_cast<const double *>(p + offsetof(TileRecs, t));
                        m.r = *reinterpret_cast<const float2 *>(p + offsetof(TileRecs, r));
                        m.v = *reinterpret_cast<const float2 *>(p + offsetof(TileRecs, v));
                        m.d = *reinterpret_cast<const float *>(p + offsetof(TileRecs, dg));
                        return m;
                    };
                    start_group();
                    e0 = e1 = e2 = -0.0f;
                    Src m = take(0);
#pragma unroll
                    for (int j = 0; j < GS; ++j) {
                        Src next = m;
                        if (j + 1 < GS)
                            next = take(j + 1);  // in flight during this step
                        float c0 = -0.0f, c1 = -0.0f, c2 = -0.0f;
                        causal_pair(m, c0, c1, c2);
                        e0 = row_rotate_f32(e0) + c0;
                        if (GRAD) {
                            if (!UNI)
                                e1 = row_rotate_f32(e1) + c1;
                            e2 = row_rotate_f32(e2) + c2;
                        }
                        m = next;
#pragma unroll
                        for (int q = 0; q < KT; ++q)
                            pin(f[q]);
                        step_end();
                    }
                    fold_back();
                    fold_trig();
                };
                if (cols) {
                    for (int sub = mlo; sub < mhi; sub += 16) {
                        // first 8 steps: lane i ends with source sub + ((i + 7) mod 16)
                        float h0, h1, h2, e0, e1, e2;
                        rotate(sub, std::integral_constant<int, 0>{}, h0, h1, h2);
                        // then with source sub + ((i + 15) mod 16), whose first-half sum is 8 lanes
                        // back; add the halves, then the four rows: row z of lanes ends with plane
                        // z (0 and 2 with the uniform background)
                        rotate(sub, std::integral_constant<int, 1>{}, e0, e1, e2);
                        double w = join_halves(h0, e0);
                        int plane = lane >> 4;
                        if (!GRAD) {
                            w = sum_rows_f64(w);
                        } else if (UNI) {
                            w = sum_rows2(w, join_halves(h2, e2));
                            plane *= 2;
                        } else {
                            const double w2 = join_halves(h2, e2);
                            w = sum_rows4(w, join_halves(h1, e1), w2, w2);
                        }
                        if (plane < CP)
                            lcol[buf][plane][wave][sub + ((li + 15) & 15)] = float(w);
                    }
                } else if (trig_only) {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, trig_pair);
                        fold_trig();
                    }
                } else if (causal) {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, [&](const Src &m) {
                            float c0 = -0.0f, c1 = -0.0f, c2 = -0.0f;
                            causal_pair(m, c0, c1, c2);  // column sums unused
                        });
                        fold_back();
                        fold_trig();
                    }
                } else {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, anti_pair);
                        fold_back();
                    }
                }
                if (causal) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        const double dn = trn[q] - last;
                        const double fn = exp(-a.omega * dn);
                        acc[q][3] += fn * gt[q][0];
                        if (GRAD) {
                            acc[q][4] += fn * gt[q][1];
                            acc[q][5] += fn * fma(dn, gt[q][0], gt[q][2]);
                        }
                    }
                }
            } else {
                // tiles overlapping the block's time range: per-pair tie-group
                // masks and the triggering time factor formed per pair in FP64
                for (int m0 = mlo; m0 < mhi; m0 += GS) {
                    float f[KT][6];
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < 6; ++z)
                            f[q][z] = -0.0f;
                    for (int j = 0; j < GS; ++j) {
                        const int m = m0 + j;
                        const double xm = T.x[m], ym = T.y[m], tm = T.t[m];
                        const float2 rm = T.r[m], um = T.u[m];
                        const float rhm = rm.x, rlm = rm.y, uhm = um.x, ulm = um.y;
                        const int gm = T.dg[m].g;
#pragma unroll
                        for (int q = 0; q < KT; ++q) {
                            float D, A, Alo = 0.0f;
                            if (UNI)
                                geom_da_uni(xn[q], yn[q], tsn[q], xm, ym, tm, D, A, Alo);
                            else
                                geom_da(xn[q], yn[q], tsn[q], xm, ym, tm, D, A);
                            const double dt = tsn[q] - tm;
                            float b = __builtin_amdgcn_exp2f(-A);
                            if (UNI)
                                b = fmaf(-LN2F * Alo, b, b);
                            b = (gm != gn[q]) ? b : 0.0f;
                            const float t1 = fmaf(rlm, D, rhm * D);
                            const float arg = float(fma(a.w2, dt, double(t1)));
                            const float E = __builtin_amdgcn_exp2f(-arg);
                            float p = fmaf(ulm, E, uhm * E);
                            p = (gm < gn[q]) ? p : 0.0f;
                            f[q][0] += b;
                            f[q][3] += p;
                            if (GRAD) {
                                if (!UNI)
                                    f[q][1] = fmaf(b, D, f[q][1]);
                                f[q][2] = fmaf(b, A, f[q][2]);
                                f[q][4] = fmaf(p, t1, f[q][4]);
                                f[q][5] = fmaf(p, float(dt), f[q][5]);
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        acc[q][0] += double(f[q][0]);
                        acc[q][3] += double(f[q][3]);
                        if (GRAD) {
                            acc[q][1] += double(f[q][1]);
                            acc[q][2] += double(f[q][2]);
                            acc[q][4] += double(f[q][4]);
                            acc[q][5] += double(f[q][5]) * a.inv_st;
                        }
                    }
                }
            }

            stage_wait();
            __syncthreads();

            if (cols && own) {
                // owner lane of source tid: the four waves' sums in a fixed order
                const int j = k * TS + tid - jb;
                double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
                for (int w = 0; w < NW; ++w) {
                    s0 += double(lcol[buf][0][w][tid]);
                    if (GRAD) {
                        if (!UNI)
                            s1 += double(lcol[buf][CP / 2][w][tid]);
                        s2 += double(lcol[buf][CP - 1][w][tid]);
                    }
                }
                pc[j] += s0 * a.out_exp;
                if (GRAD) {
                    if (!UNI)
                        pc[cstride + j] += s1 * (a.out_s1 * a.out_exp);
                    pc[2 * cstride + j] += (s2 - s1) * (a.out_s2 * a.out_exp);
                }
            }
        }

        // this block's row sums against the column group, in the sums' natural units
        double *out = a.srow + int64_t(slot) * (GRAD ? 6 : 2) * stride;
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            if (i >= iend)
                continue;
            const int rr = i - a.row_begin - rb0;
            const double ce = a.out_exp;
            out[0 * stride + rr] = acc[q][0] * ce;
            out[(GRAD ? 3 : 1) * stride + rr] = acc[q][3] * ce;
            if (GRAD) {
                out[1 * stride + rr] = acc[q][1] * (a.out_s1 * ce);
                out[2 * stride + rr] = (acc[q][2] - acc[q][1]) * (a.out_s2 * ce);
                out[4 * stride + rr] = acc[q][4] * (a.out_g1 * ce);
                out[5 * stride + rr] = acc[q][5] * ce;
            }
        }
    }
}

// ------------------------------------------------ several theta in one sweep
//
// The forward-only FP32 sweep for NT parameter vectors at once (S0 and G0 of
// each), on the same events and the same work decomposition as k_pair_f32.
// What the vectors share is computed once per pair: the pair differences and
// the squared distance d2 in FP64 and, for vectors after the first, the
// squared time difference.  Positions and times are scaled for theta 0; for
// theta k the squared distance in its own scale is d2 cx_k and the background
// exponent A_k = d2 cx_k + dt^2 ct_k (cx_k = (sx_k / sx_0)^2,
// ct_k = (st_k / st_0)^2), each formed in FP64 and rounded once to FP32, so
// that every FP32 value of theta k is the one a single sweep at theta k forms
// (up to FP64 rounding).  Per-theta source fields: r_m and v_m (hi, lo);
// u_m, the time offsets and tie groups are shared.
// Theta k's row sums go to row planes k (S0) and NT + k (G0) of a slot and its
// column sums to column plane k.

struct PairBatchF32 {
    const double *xs, *ys, *tsd, *t;  // positions and times scaled for theta 0
    const float2 *r2, *v2;            // theta k's (hi, lo) fields at r2 + k * theta_stride
    const float2 *u2;                 // (hi, lo) of u_m
    const DeltaGroup *dg;
    const int *g;
    const double *tile;
    const int *kstrict, *kend;
    CellMap cells;
    double *srow, *scol;  // slots as in PairF32
    int ge;
    int row_begin, row_end, rows_pad, num_tiles, num_tb;
    int rr, cg;
    int sym, trig_cull;
    int theta_stride;
    // (sx_k / sx_0)^2 and (st_k / st_0)^2: theta k's spatial and temporal scales against theta 0's
    double cx[MAX_FUSED_THETA], ct2[MAX_FUSED_THETA], omega[MAX_FUSED_THETA], w2[MAX_FUSED_THETA];
    double out_exp;
};

template <int NT, bool UNI>
__global__ __launch_bounds__(WG) HK_WAVES(HAWKES_WAVES_GRAD) void k_pair_f32_batch(PairBatchF32 a)
{
    static_assert(NT >= 1 && NT <= MAX_FUSED_THETA, "fused theta count");
    struct alignas(16) TileRecs {
        double x[TS], y[TS], t[TS];
        float2 r[NT][TS], v[NT][TS], u[TS];
        DeltaGroup dg[TS];
    };
    __shared__ TileRecs lt2[2];
    __shared__ float lcol[2][NT][NW][TS];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15;
    int gr, gc, slot;
    if (!map_cell(a.cells, blockIdx.x, gr, gc, slot))
        return;
    const int b_first = gr * a.rr;
    const int b_stop = (b_first + a.rr < a.num_tb) ? b_first + a.rr : a.num_tb;
    // sources [jb, js) of the column group: tiles [kg0, kg1), of each the sources [mlo, mhi)
    const int jb = gc * a.cg, js = (jb + a.cg < a.num_tiles * TS) ? jb + a.cg : a.num_tiles * TS;
    const int kg0 = jb / TS, kg1 = (js + TS - 1) / TS;
    const int mlo = jb & (TS - 1), mhi = (a.cg < TS) ? mlo + a.cg : TS;
    const bool own = tid >= mlo && tid < mhi;  // this lane's source of a tile is in the group
    const int64_t stride = a.ge;
    const int rb0 = b_first * TB;
    const int64_t cstride = a.cg;
    double *pc = a.scol + int64_t(slot) * NT * cstride;
    if (a.sym && own) {
        for (int k = kg0; k < kg1; ++k)
#pragma unroll
            for (int z = 0; z < NT; ++z)
                pc[z * cstride + k * TS + tid - jb] = 0.0;
    }

    auto stage = [&](int k, int buf) {
        TileRecs &T = lt2[buf];
        int o = tid;
        asm volatile("" : "+v"(o));
        const int wb = tid & ~63;
        auto copy = [&](const void *src, void *dst) {
            const unsigned *s = reinterpret_cast<const unsigned *>(src);
            unsigned *d = reinterpret_cast<unsigned *>(dst);
            lds_dma4(s + o, d + wb);
            lds_dma4(s + TS + o, d + TS + wb);
        };
        copy(a.xs + k * TS, T.x);
        copy(a.ys + k * TS, T.y);
        copy(a.tsd + k * TS, T.t);
#pragma unroll
        for (int z = 0; z < NT; ++z) {
            copy(a.r2 + int64_t(z) * a.theta_stride + k * TS, T.r[z]);
            copy(a.v2 + int64_t(z) * a.theta_stride + k * TS, T.v[z]);
        }
        copy(a.u2 + k * TS, T.u);
        copy(a.dg + k * TS, T.dg);
    };

    const Rotation rot(li);

    for (int b = b_first; b < b_stop; ++b) {
        const int i0 = a.row_begin + b * TB;
        const int iend = (i0 + TB < a.row_end) ? i0 + TB : a.row_end;
        int k0 = kg0;
        int skip_gap = INT_MAX;  // gaps as the bits of a float >= 0, ordered like it, in scalar registers
        // the gap that the sums of tile k's own events ask for (symmetric sweep: they take column sums)
        auto tile_gap = [&](int k) { return a.sym ? tile_word(a.tile, k & ~(KT - 1)).gap_bits() : 0; };
        if (a.trig_cull) {
            const TileWord w = tile_word(a.tile, KT * b);
            skip_gap = w.gap_bits();
            k0 = (kg0 > w.klo) ? kg0 : w.klo;
            k0 = (k0 < a.num_tiles) ? k0 : a.num_tiles - 1;
        } else {
            stage(k0, 0);
        }
        const double t_lo = a.t[i0], t_hi = a.t[iend - 1];

        double xn[KT], yn[KT], tsn[KT], trn[KT];
        int gn[KT];
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            const bool in = i < iend;
            xn[q] = in ? a.xs[i] : PAD_COORD;
            yn[q] = in ? a.ys[i] : PAD_COORD;
            tsn[q] = in ? a.tsd[i] : PAD_TIME;
            trn[q] = a.t[in ? i : iend - 1];
            gn[q] = in ? a.g[i] : INT_MAX;
        }
        double acc[KT][NT][2];
#pragma unroll
        for (int q = 0; q < KT; ++q)
#pragma unroll
            for (int z = 0; z < NT; ++z)
                acc[q][z][0] = acc[q][z][1] = 0.0;

        const int k_strict = a.kstrict[b], k_end = a.kend[b];
        const int k1 = (kg1 < k_end) ? kg1 : k_end;
        if (a.trig_cull && k0 < k1)
            stage(k0, 0);
        stage_wait();
        __syncthreads();

        double next_first = a.tile[3 * k0 + 0], next_last = a.tile[3 * k0 + 1];
        int next_gap = a.trig_cull ? tile_gap(k0) : 0;
        for (int k = k0; k < k1; ++k) {
            const int buf = (k - k0) & 1;
            const double first = next_first, last = next_last;
            const int gap = skip_gap > next_gap ? skip_gap : next_gap;
            if (k + 1 < k1) {
                stage(k + 1, buf ^ 1);
                next_first = a.tile[3 * k + 3];
                next_last = a.tile[3 * k + 4];
                if (a.trig_cull)
                    next_gap = tile_gap(k + 1);
            }

            const int cls = (last < t_lo) ? CAUSAL : ((first > t_hi) ? ANTI : MIXED);
            const bool trig_only = (cls == CAUSAL) && a.trig_cull && (t_lo - last > double(__int_as_float(gap)));
            const bool cols = (k < k_strict) && !trig_only;

            double gt[KT][NT];
#pragma unroll
            for (int q = 0; q < KT; ++q)
#pragma unroll
                for (int z = 0; z < NT; ++z)
                    gt[q][z] = 0.0;

            const TileRecs &T = lt2[buf];

            // Per pair: each vector's squared distance in its own spatial scale,
            // d2 cx_z in FP64 rounded once to FP32 (so that its triggering exponent
            // r_m D is rounded as a single sweep at that vector rounds it), and its
            // background term.
            auto pair_terms = [&](double xn_, double yn_, double tn_, double xm, double ym, double tm,
                                  float (&Dz)[NT], float (&bz)[NT]) {
                const double dx = xn_ - xm, dy = yn_ - ym, dt = tn_ - tm;
                const double d2 = fma(dy, dy, dx * dx);
                const double dt2 = dt * dt;
#pragma unroll
                for (int z = 0; z < NT; ++z) {
                    const double dz = (z == 0) ? d2 : d2 * a.cx[z];
                    Dz[z] = float(dz);
                    if (UNI) {
                        const double a2 = (z == 0) ? dt2 : dt2 * a.ct2[z];
                        const float A = float(a2), Alo = float(a2 - double(A));
                        const float e = __builtin_amdgcn_exp2f(-A);
                        bz[z] = fmaf(-LN2F * Alo, e, e);
                    } else {
                        const float A = (z == 0) ? float(fma(dt, dt, d2)) : float(fma(dt2, a.ct2[z], dz));
                        bz[z] = __builtin_amdgcn_exp2f(-A);
                    }
                }
            };
            // squared distances only (triggering terms of tiles without background terms)
            auto dist_terms = [&](double xn_, double yn_, double xm, double ym, float (&Dz)[NT]) {
                const double dx = xn_ - xm, dy = yn_ - ym;
                const double d2 = fma(dy, dy, dx * dx);
#pragma unroll
                for (int z = 0; z < NT; ++z)
                    Dz[z] = float((z == 0) ? d2 : d2 * a.cx[z]);
            };

            if (cls != MIXED) {
                const bool causal = (cls == CAUSAL);
                const char *lbase = reinterpret_cast<const char *>(&lt2[0]);
                const int tbase = buf * int(sizeof(TileRecs));
                struct Src {
                    double x, y, t;
                    float2 r[NT], v[NT];
                };
                float f[KT][2 * NT];  // S0 of each vector, then G0
                auto start_group = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < 2 * NT; ++z)
                            f[q][z] = -0.0f;
                };
                auto pin_sums = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q)
                        pin(f[q]);
                    step_end();
                };
                auto fold_back = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            acc[q][z][0] += double(f[q][z]);
                };
                auto fold_trig = [&]() {
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            gt[q][z] += double(f[q][NT + z]);
                };
                // background + triggering terms of one source for the lane's targets;
                // adds each vector's background terms over those targets to c[z]
                auto causal_pair = [&](const Src &m, float (&c)[NT]) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float Dz[NT], bz[NT];
                        pair_terms(xn[q], yn[q], tsn[q], m.x, m.y, m.t, Dz, bz);
#pragma unroll
                        for (int z = 0; z < NT; ++z) {
                            const float D = Dz[z];
                            const float t1 = fmaf(m.r[z].y, D, m.r[z].x * D);
                            const float E = __builtin_amdgcn_exp2f(-t1);
                            const float p = fmaf(m.v[z].y, E, m.v[z].x * E);
                            f[q][z] += bz[z];
                            f[q][NT + z] += p;
                            c[z] += bz[z];
                        }
                    }
                };
                auto trig_pair = [&](const Src &m) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float Dz[NT];
                        dist_terms(xn[q], yn[q], m.x, m.y, Dz);
#pragma unroll
                        for (int z = 0; z < NT; ++z) {
                            const float D = Dz[z];
                            const float t1 = fmaf(m.r[z].y, D, m.r[z].x * D);
                            const float E = __builtin_amdgcn_exp2f(-t1);
                            f[q][NT + z] += fmaf(m.v[z].y, E, m.v[z].x * E);
                        }
                    }
                };
                auto anti_pair = [&](const Src &m) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        float Dz[NT], bz[NT];
                        pair_terms(xn[q], yn[q], tsn[q], m.x, m.y, m.t, Dz, bz);
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            f[q][z] += bz[z];
                    }
                };
                auto field = [&](const char *p, size_t off, int z) {
                    return *reinterpret_cast<const float2 *>(p + off + z * sizeof(float2) * TS);
                };
                auto load = [&](const char *p) {
                    Src m;
                    m.x = *reinterpret_cast<const double *>(p + offsetof(TileRecs, x));
                    m.y = *reinterpret_cast<const double *>(p + offsetof(TileRecs, y));
                    m.t = *reinterpret_cast<const double *>(p + offsetof(TileRecs, t));
#pragma unroll
                    for (int z = 0; z < NT; ++z) {
                        m.r[z] = field(p, offsetof(TileRecs, r), z);
                        m.v[z] = field(p, offsetof(TileRecs, v), z);
                    }
                    return m;
                };
                // a group of 8 sources in order, the same for every lane
                auto in_order = [&](int m0, auto &&pair) {
                    const char *g0 = lbase + (tbase + m0 * 8);
                    start_group();
                    Src m = load(g0);
#pragma unroll
                    for (int j = 0; j < GS; ++j) {
                        Src next = m;
                        if (j + 1 < GS)
                            next = load(g0 + 8 * (j + 1));  // in flight during this step
                        pair(m);
                        m = next;
                        pin_sums();
                    }
                };
                // 8 steps of the 16-source rotation, as in k_pair_f32
                auto rotate = [&](int sub, auto half, float (&e)[NT]) {
                    constexpr int HALF = decltype(half)::value;
                    const int base = tbase + sub * 8;
                    start_group();
#pragma unroll
                    for (int z = 0; z < NT; ++z)
                        e[z] = -0.0f;
                    Src m = load(lbase + rot.at(0, 64 * HALF, base));
#pragma unroll
                    for (int j = 0; j < GS; ++j) {
                        Src next = m;
                        if (j + 1 < GS)
                            next = load(lbase + rot.at(j + 1, 64 * HALF, base));
                        float c[NT];
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            c[z] = -0.0f;
                        causal_pair(m, c);
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            e[z] = row_rotate_f32(e[z]) + c[z];
                        m = next;
                        pin_sums();
                    }
                    fold_back();
                    fold_trig();
                };
                if (cols) {
                    for (int sub = mlo; sub < mhi; sub += 16) {
                        float h[NT], e[NT];
                        rotate(sub, std::integral_constant<int, 0>{}, h);
                        rotate(sub, std::integral_constant<int, 1>{}, e);
                        // row z of lanes ends with vector z's sums over the four rows
                        static_assert(NT == 2, "one swap serves two vectors");
                        const double w = sum_rows2(join_halves(h[0], e[0]), join_halves(h[1], e[1]));
                        const int z = lane >> 4;
                        if (z < NT)
                            lcol[buf][z][wave][sub + ((li + 15) & 15)] = float(w);
                    }
                } else if (trig_only) {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, trig_pair);
                        fold_trig();
                    }
                } else if (causal) {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, [&](const Src &m) {
                            float c[NT] = {-0.0f, -0.0f};  // column sums unused
                            causal_pair(m, c);
                        });
                        fold_back();
                        fold_trig();
                    }
                } else {
                    for (int m0 = mlo; m0 < mhi; m0 += GS) {
                        in_order(m0, anti_pair);
                        fold_back();
                    }
                }
                if (causal) {
#pragma unroll
                    for (int q = 0; q < KT; ++q) {
                        const double dn = trn[q] - last;
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            acc[q][z][1] += exp(-a.omega[z] * dn) * gt[q][z];
                    }
                }
            } else {
                // tiles overlapping the block's time range: tie-group masks and the
                // triggering time factor per pair in FP64
                for (int m0 = mlo; m0 < mhi; m0 += GS) {
                    float f[KT][NT][2];
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < NT; ++z)
                            f[q][z][0] = f[q][z][1] = -0.0f;
#pragma unroll 1
                    for (int j = 0; j < GS; ++j) {
                        const int m = m0 + j;
                        const double xm = T.x[m], ym = T.y[m], tm = T.t[m];
                        const float2 um = T.u[m];
                        const int gm = T.dg[m].g;
#pragma unroll
                        for (int q = 0; q < KT; ++q) {
                            float Dz[NT], bz[NT];
                            pair_terms(xn[q], yn[q], tsn[q], xm, ym, tm, Dz, bz);
                            const double dt = tsn[q] - tm;
#pragma unroll
                            for (int z = 0; z < NT; ++z) {
                                const float2 rm = T.r[z][m];
                                const float D = Dz[z];
                                const float b = (gm != gn[q]) ? bz[z] : 0.0f;
                                const float t1 = fmaf(rm.y, D, rm.x * D);
                                const float arg = float(fma(a.w2[z], dt, double(t1)));
                                const float E = __builtin_amdgcn_exp2f(-arg);
                                const float p = fmaf(um.y, E, um.x * E);
                                f[q][z][0] += b;
                                f[q][z][1] += (gm < gn[q]) ? p : 0.0f;
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < KT; ++q)
#pragma unroll
                        for (int z = 0; z < NT; ++z) {
                            acc[q][z][0] += double(f[q][z][0]);
                            acc[q][z][1] += double(f[q][z][1]);
                        }
                }
            }

            stage_wait();
            __syncthreads();

            if (cols && own) {
                const int j = k * TS + tid - jb;
#pragma unroll
                for (int z = 0; z < NT; ++z) {
                    double s = 0.0;
#pragma unroll
                    for (int w = 0; w < NW; ++w)
                        s += double(lcol[buf][z][w][tid]);
                    pc[z * cstride + j] += s * a.out_exp;
                }
            }
        }

        double *out = a.srow + int64_t(slot) * 2 * NT * stride;
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            if (i >= iend)
                continue;
            const int rr = i - a.row_begin - rb0;
#pragma unroll
            for (int z = 0; z < NT; ++z) {
                out[z * stride + rr] = acc[q][z][0] * a.out_exp;
                out[(NT + z) * stride + rr] = acc[q][z][1] * a.out_exp;
            }
        }
    }
}

// What the host cannot know about a call's events, worked out by one
// workgroup: the status words (data checks, largest u_m, empty rescue lists),
// which tiles each target block b of the sweep visits, and, for the symmetric
// sweep, the cells.
//   Tiles: [klo, kend[b]), of which those before kstrict[b] lie strictly before the
// block in time and take column sums (symmetric sweep: whole blocks; row
// sweep: none).  Symmetric sweep: from kend on lie the blocks whose first
// time is above b's last.  With trig_cull (skip mode) klo (tile_word of tile
// KT b) is the first tile within the triggering range of the block, with the
// block's gap; in the row sweep kend then leaves out the tiles more than that
// gap after it.
//   Cells: row group gr reaches the column groups up to gchi[gr] (the last of its
// blocks' kend) from gclo[gr] on (the least klo of its and later blocks); its cells are
// numbered from rowstart[gr] on, latest row groups first (rowstart[num_gr - 1]
// = 0), and *total is their number.
struct PlanArgs {
    const StageBlock *blocks;
    int num_blocks;
    int *status;
    const double *t;
    double *tile;
    int64_t n, num_tb, row_begin, row_end;
    int num_tiles;
    int sym, trig_cull;
    double skip_gap, omega;
    const RateBound *bounds;  // null: none, every gap is skip_gap
    double min_span;
    double *far_trig, *reach;  // [tile], with bounds
    int rr, cg, num_gr;
    int *kstrict, *kend, *gchi, *gclo, *rowstart, *total;
};

constexpr int PLAN_WG = 1024;
static_assert(MAX_SYM_GROUPS <= PLAN_WG, "one row group per thread");

// Smallest bounds over the rows [i0, i1).
__device__ inline RateBound rows_bound(const RateBound *bounds, int64_t i0, int64_t i1)
{
    RateBound v = {HUGE_VALF, HUGE_VALF, 0.0f};
    for (int64_t g = i0 / BOUND_ROWS; g <= (i1 - 1) / BOUND_ROWS; ++g) {
        v.bg = fminf(v.bg, bounds[g].bg);
        v.trig = fminf(v.trig, bounds[g].trig);
    }
    return v;
}

// A gap in a TileWord: rounded up.
__device__ inline float gap_word(double gap)
{
    const float f = float(gap);
    return double(f) < gap ? nextafterf(f, HUGE_VALF) : f;
}

// With the rows' bounds (skip mode): each block's gap, beyond which all n background terms
// together are below 2^-RATE_BITS of its rows' rates, in its TileWord, and two
// nondecreasing functions of the tile k that first_tile_needed searches:
//   far_trig[k]  log2 of sum_{m in tiles 0..k} u_m exp(-omega (t_0 - t_m)), t_m taken
//                as its tile's last time: the sources' part of their triggering terms;
//   reach[k]     the largest last time, in the symmetric sweep plus own gap, of tiles 0..k.
// Both are prefix combinations over the tiles: a chunk of tiles per thread, a scan over the
// threads (exponentials in FP32: 1e-5 of a bit).
__device__ inline void plan_ranges(const PlanArgs &a)
{
    __shared__ double sum[PLAN_WG / 64], time[PLAN_WG / 64], far[PLAN_WG / 64];
    const int tid = threadIdx.x;
    for (int64_t b = tid; b < a.num_tb; b += PLAN_WG) {
        const int64_t i0 = a.row_begin + b * TB, i1 = i0 + TB < a.row_end ? i0 + TB : a.row_end;
        const double need = RATE_BITS + log2(double(a.n)) - double(rows_bound(a.bounds, i0, i1).bg);
        const double gap = !(need < SKIP_EXPONENT) ? a.skip_gap
                                                   : a.skip_gap * sqrt(fmax(need, 0.0) / SKIP_EXPONENT);
        *reinterpret_cast<TileWord *>(a.tile + 3 * (KT * b) + 2) = TileWord{0, gap_word(gap)};
    }
    __syncthreads();
    const int per = (a.num_tiles + PLAN_WG - 1) / PLAN_WG;
    const int k0 = tid * per < a.num_tiles ? tid * per : a.num_tiles;
    const int k1 = k0 + per < a.num_tiles ? k0 + per : a.num_tiles;
    const float w = float(a.omega * LOG2E);
    auto decay = [&](double days) { return double(exp2f(-w * float(days))); };
    // sum over tiles up to k in units of the tile's last time, and the largest reach
    auto extend = [&](double &v, double &t, double &r, int k) {
        const double last = a.tile[3 * k + 1];
        constexpr int PER_TILE = TS / BOUND_ROWS;
        const int groups = int((a.n + BOUND_ROWS - 1) / BOUND_ROWS);
        double u = 0.0;
        for (int g = k * PER_TILE; g < (k + 1) * PER_TILE && g < groups; ++g)
            u += double(a.bounds[g].usum);
        v = v * decay(last - t) + u;
        t = last;
        r = fmax(r, a.sym ? last + double(tile_word(a.tile, k & ~(KT - 1)).gap) : last);
    };
    const double t_chunk = a.tile[3 * (k0 < a.num_tiles ? k0 : a.num_tiles - 1) + 1];
    double v = 0.0, t = t_chunk, r = -HUGE_VAL;
    for (int k = k0; k < k1; ++k)
        extend(v, t, r, k);
    // inclusive over the wave's lanes, then over the waves
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double pv = __shfl_up(v, o), pt = __shfl_up(t, o), pr = __shfl_up(r, o);
        if (lane >= o) {
            v += pv * decay(t - pt);
            r = fmax(r, pr);
        }
    }
    if (lane == 63) {
        sum[wave] = v;
        time[wave] = t;
        far[wave] = r;
    }
    __syncthreads();
    double av = 0.0, at = wave > 0 ? time[0] : t_chunk, ar = -HUGE_VAL;  // over the earlier waves
    for (int z = 0; z < wave; ++z) {
        av = av * decay(time[z] - at) + sum[z];
        at = time[z];
        ar = fmax(ar, far[z]);
    }
    double pv = __shfl_up(v, 1), pt = __shfl_up(t, 1), pr = __shfl_up(r, 1);
    if (lane == 0) {
        pv = av;
        pt = at;
        pr = ar;
    } else {
        if (wave > 0)  // the first wave has none before it, and pt may lie far before t_chunk
            pv += av * decay(pt - at);
        pr = fmax(pr, ar);
    }
    const double t_first = a.tile[1];
    for (int k = k0; k < k1; ++k) {
        extend(pv, pt, pr, k);
        a.far_trig[k] = double(log2f(float(pv))) + double(w) * (pt - t_first);
        a.reach[k] = pr;
    }
    __syncthreads();
}

// First tile the block of rows [i0, i1) that starts at t0 visits: from there on triggering terms
// matter to its rows, background terms to its rows (its own gap) or to the tile's (their reach, in the
// symmetric sweep), and all is within the triggering range.  Each condition is monotone in the tile.
__device__ inline int first_tile_needed(const PlanArgs &a, int64_t i0, int64_t i1, double t0, double gap, double range)
{
    const double limit = double(rows_bound(a.bounds, i0, i1).trig) - RATE_BITS +
                         double(float(a.omega * LOG2E)) * (t0 - a.tile[1]);
    int lo = 0, hi = a.num_tiles;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const double last = a.tile[3 * mid + 1];
        if (last < t0 - range || (last < t0 - gap && a.reach[mid] < t0 && a.far_trig[mid] < limit))
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

__device__ __forceinline__ void plan(const PlanArgs &a, double umax, int flags)
{
    __shared__ int scan[PLAN_WG];
    const int tid = threadIdx.x;
    if (tid == 0) {
        a.status[0] = flags;
        reinterpret_cast<double *>(a.status)[STATUS_UMAX] = umax;
    }
    if (tid < 2 * MAX_FUSED_THETA)
        a.status[STATUS_RESCUE + tid] = 0;
    const double gap = a.trig_cull ? trig_cull_gap(umax, a.omega, a.skip_gap) : 0.0;
    const bool bounded = a.trig_cull && a.bounds && a.t[a.n - 1] - a.t[0] > a.min_span;
    if (bounded)
        plan_ranges(a);

    auto first_t = [&](int64_t c) { return a.t[c * TB]; };
    auto last_t = [&](int64_t c) { return a.t[((c + 1) * TB < a.n ? (c + 1) * TB : a.n) - 1]; };
    // a block's neighbours settle its bounds unless a tie run crosses into them
    auto first_at_or_after = [&](int64_t b) {
        const double tl = first_t(b);
        if (b == 0 || last_t(b - 1) < tl)
            return b;
        int64_t lo = 0, hi = b;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (last_t(mid) < tl)
                lo = mid + 1;
            else
                hi = mid;
        }
        return lo;
    };
    auto first_after = [&](int64_t b) {
        const double th = last_t(b);
        if (b + 1 == a.num_tb || first_t(b + 1) > th)
            return b + 1;
        int64_t lo = b + 1, hi = a.num_tb;
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (first_t(mid) > th)
                hi = mid;
            else
                lo = mid + 1;
        }
        return lo;
    };
    auto tile_end = [&](int64_t b) {
        const int64_t e = KT * first_after(b);
        return int(e < a.num_tiles ? e : int64_t(a.num_tiles));
    };
    for (int64_t b = tid; b < a.num_tb; b += PLAN_WG) {
        const int64_t i0 = a.row_begin + b * TB, i1 = i0 + TB < a.row_end ? i0 + TB : a.row_end;
        int strict = 0, end = a.num_tiles;
        double block_gap = a.skip_gap;
        if (a.trig_cull) {
            const double t0 = a.t[i0];
            if (bounded)
                block_gap = tile_word(a.tile, int(KT * b)).gap;
            const int klo = bounded ? first_tile_needed(a, i0, i1, t0, block_gap, gap)
                                    : first_tile_within(a.tile, a.num_tiles, t0, gap);
            *reinterpret_cast<TileWord *>(a.tile + 3 * (KT * b) + 2) = TileWord{klo, gap_word(block_gap)};
        }
        if (a.sym) {
            strict = int(KT * first_at_or_after(b));
            end = tile_end(b);
        } else if (a.trig_cull) {
            end = first_tile_after(a.tile, a.num_tiles, a.t[i1 - 1], block_gap);
        }
        a.kstrict[b] = strict;
        a.kend[b] = end;
    }
    if (!a.sym)
        return;
    // a group's first tile: the least of its blocks' and, so that gclo is nondecreasing, of the later groups'.
    // Where the data checks failed it is 0: with unsorted times gchi need not be nondecreasing, and
    // k_fold's cells of a column then fall with the row group only if gclo is 0 throughout
    const bool cull = a.trig_cull && !flags;
    int first = a.num_tiles;
    if (cull) {
        __syncthreads();  // the blocks' words
        if (tid < a.num_gr)
            for (int64_t b = int64_t(tid) * a.rr; b < a.num_tb && b < int64_t(tid + 1) * a.rr; ++b) {
                const int klo = tile_word(a.tile, int(KT * b)).klo;
                first = klo < first ? klo : first;
            }
        scan[tid] = first;
        __syncthreads();
        for (int o = 1; o < PLAN_WG; o <<= 1) {
            if (o >= a.num_gr)
                break;
            const int v = (tid + o < PLAN_WG) ? scan[tid + o] : a.num_tiles;
            __syncthreads();
            scan[tid] = first = v < first ? v : first;
            __syncthreads();
        }
    }
    int cells = 0;
    if (tid < a.num_gr) {
        const int64_t bf = int64_t(tid) * a.rr;
        const int64_t bl = (bf + a.rr < a.num_tb ? bf + a.rr : a.num_tb) - 1;
        const int hi = int((int64_t(tile_end(bl)) * TS + a.cg - 1) / a.cg) - 1;
        int lo = 0;
        if (cull) {
            lo = int(int64_t(first) * TS / a.cg);
            lo = lo < hi ? lo : hi;
        }
        a.gchi[tid] = hi;
        a.gclo[tid] = lo;
        cells = hi - lo + 1;
    }
    // first cells: sums of the later row groups' cell counts
    __syncthreads();
    scan[tid] = cells;
    __syncthreads();
    for (int o = 1; o < PLAN_WG; o <<= 1) {
        if (o >= a.num_gr)
            break;
        const int v = (tid + o < PLAN_WG) ? scan[tid + o] : 0;
        __syncthreads();
        scan[tid] += v;
        __syncthreads();
    }
    if (tid < a.num_gr)
        a.rowstart[tid] = scan[tid] - cells;
    if (tid == 0)
        *a.total = scan[0];
}

__global__ __launch_bounds__(PLAN_WG) void k_plan(PlanArgs a)
{
    double u = 0.0;
    int flags = 0;
    for (int b = threadIdx.x; b < a.num_blocks; b += PLAN_WG) {
        u = fmax(u, a.blocks[b].umax);
        flags |= int(a.blocks[b].flags);
    }
    join_stage<PLAN_WG / 64>(u, flags);
    plan(a, u, flags);
}

// Staging and plan in one workgroup, for few events (a launch less).
constexpr int64_t STAGE_PLAN_EVENTS = 4096;
template <bool F32>
__global__ __launch_bounds__(PLAN_WG) void k_stage_plan(StageArgs s, PlanArgs a)
{
    double u = 0.0;
    int flags = 0;
    for (int64_t i = threadIdx.x; i < s.n_pad; i += PLAN_WG)
        stage_event<F32>(s, i, u, flags);
    join_stage<PLAN_WG / 64>(u, flags);  // its barrier also publishes the tile records
    plan(a, u, flags);
}

struct PairF64 {
    const double *t, *x, *y, *s;
    const int *g;
    const double *tile;
    const int *kstrict, *kend;  // as in PairF32
    CellMap cells;
    double *srow, *scol;     // slots as in PairF32
    int ge;
    int n, row_begin, row_end, rows_pad, num_tiles, num_tb;
    int rr, cg, sym;
    double ax, at, qh, omega;  // log2(e) times: 1/(2 tau_x^2), 1/(2 tau_t^2), 1/(2 h0^2), omega
    double out_g1;             // 1 / qh
};

// 2^y for y <= 0 in FP64 (the pair terms of the FP64 sweep, whose exponents are
// formed in units of log2): y = n/16 + r with n = rint(16 y) and |r| <= 1/32,
// 2^y = 2^(n >> 4) T_j (1 + d_j + r P(r)), j = n & 15, where T_j is 2^(j/16) rounded to
// FP64 and d_j what that rounding left out (relative), so that only the last
// fma and the scaling round at full size (0.66 ulp at worst, just below a power of two).  P is the degree-5
// interpolant of (2^r - 1)/r at the Chebyshev nodes of [-1/32, 1/32] (error of
// 2^r below 1.5e-17 relative).  n comes from the low word of 16 y + 1.5 2^52.
// 11 FP64 operations where a degree-12 polynomial over |r| <= 1/2 took 17.  The 16
// entries of T (and of d) span the LDS banks once: lanes read any of them
// without conflict.  Exponents below -2000 give 0.
constexpr int EXP2_TABLE = 16;
__device__ const double exp2_table_init[2 * EXP2_TABLE] = {
    0x1.0000000000000p+0,   0x1.0b5586cf9890fp+0,   0x1.172b83c7d517bp+0,   0x1.2387a6e756238p+0,
    0x1.306fe0a31b715p+0,   0x1.3dea64c123422p+0,   0x1.4bfdad5362a27p+0,   0x1.5ab07dd485429p+0,
    0x1.6a09e667f3bcdp+0,   0x1.7a11473eb0187p+0,   0x1.8ace5422aa0dbp+0,   0x1.9c49182a3f090p+0,
    0x1.ae89f995ad3adp+0,   0x1.c199bdd85529cp+0,   0x1.d5818dcfba487p+0,   0x1.ea4afa2a490dap+0,
    0x0.0p+0,               0x1.79aa65d837b6dp-54,  -0x1.01b15eaa59348p-55, 0x1.68efde3a8a894p-54,
    0x1.34d754db0abb6p-55,  0x1.59f48a72a4c6dp-55,  0x1.690cebb7aafb0p-56,  0x1.063e1e21c5409p-54,
    -0x1.3b3efbf5e2228p-54, -0x1.b32dcb94da51dp-56, 0x1.db72fc1f0eab4p-55,  0x1.1affc2b91ce27p-56,
    0x1.c1a7792cb3387p-55,  0x1.36eae30af0cb3p-56,  0x1.4a385a63d07a7p-56,  -0x1.ff7128fd391f0p-55,
};
__device__ __forceinline__ double exp2_nonpos(double y, const double *table)
{
    constexpr double MAGIC = 0x1.8p52;
    y = fmax(y, -2000.0);
    const double z = fma(y, double(EXP2_TABLE), MAGIC);
    const double r = fma(z - MAGIC, -1.0 / EXP2_TABLE, y);
    const int n = int(unsigned((unsigned long long)__double_as_longlong(z)));
    const double *e = table + (n & (EXP2_TABLE - 1));
    double q = 0x1.430a1d08ec681p-13;
    q = fma(q, r, 0x1.5d897e525c216p-10);
    q = fma(q, r, 0x1.3b2ab6fb41213p-7);
    q = fma(q, r, 0x1.c6b08d6f2a289p-5);
    q = fma(q, r, 0x1.ebfbdff82c590p-3);
    q = fma(q, r, 0x1.62e42fefa39f3p-1);
    q = fma(q, r, e[EXP2_TABLE]);
    return ldexp(fma(e[0], q, e[0]), n >> 4);
}

template <int CTRL>
__device__ __forceinline__ double dpp_mov_f64(double v)
{
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    const int lo = dpp_mov<CTRL>(int(unsigned(u))), hi = dpp_mov<CTRL>(int(unsigned(u >> 32)));
    return make_f64(unsigned(lo), unsigned(hi));
}
__device__ __forceinline__ double row_rotate_f64(double v) { return dpp_mov_f64<DPP_ROW_ROR15>(v); }

// The FP64 sweep: every pair term in FP64 with the direct formulas, on the
// same work decomposition as the FP32 sweep (row groups x column groups; over
// the whole event set the symmetric sweep, with the background column sums of
// a strictly earlier tile carried by the 16-lane rotation in FP64, summed over
// the 4 rows and the 4 waves and added to this row group's column partials).
// Bound: FP64 VALU issue: 45 FP64 operations of 61 VALU instructions per pair in
// the column loop with the gradient.  At 30,011 events 1013 -> 761 us and at 10^5
// 10.3 -> 7.8 ms against the previous loop (62 FP64 operations, a longer
// exponential and a product per sum), the value alone 875 -> 630 us.
template <bool GRAD>
__global__ __launch_bounds__(WG) HK_WAVES(GRAD ? 3 : 4) void k_pair_f64(PairF64 a)
{
    // source records as 8-byte fields (q: u_m qh), so that one rotated index addresses all
    struct TileRecs {
        double x[TS], y[TS], t[TS], u[TS], q[TS];
        int g[TS];
    };
    constexpr int CP = GRAD ? 3 : 1;
    __shared__ TileRecs lt2[2];
    __shared__ double lcol[CP][NW][TS];  // per-wave column sums of the tile just swept
    __shared__ double ltab[2 * EXP2_TABLE];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15;
    int gr, gc, slot;
    if (!map_cell(a.cells, blockIdx.x, gr, gc, slot))
        return;
    if (tid < 2 * EXP2_TABLE)
        ltab[tid] = exp2_table_init[tid];  // published by the first barrier below
    const int b_first = gr * a.rr;
    const int b_stop = (b_first + a.rr < a.num_tb) ? b_first + a.rr : a.num_tb;
    // sources [jb, js) of the column group: tiles [kg0, kg1), of each the sources [mlo, mhi)
    const int jb = gc * a.cg, js = (jb + a.cg < a.num_tiles * TS) ? jb + a.cg : a.num_tiles * TS;
    const int kg0 = jb / TS, kg1 = (js + TS - 1) / TS;
    const int mlo = jb & (TS - 1), mhi = (a.cg < TS) ? mlo + a.cg : TS;
    const bool own = tid >= mlo && tid < mhi;  // this lane's source of a tile is in the group
    const int64_t stride = a.ge;
    const int rb0 = b_first * TB;
    const int64_t cstride = a.cg;
    double *pc = a.scol + int64_t(slot) * CP * cstride;
    if (a.sym && own) {
        for (int k = kg0; k < kg1; ++k)
#pragma unroll
            for (int z = 0; z < CP; ++z)
                pc[z * cstride + k * TS + tid - jb] = 0.0;
    }

    struct Fetched {
        double x, y, t, u;
        int g;
    };
    auto fetch = [&](int j) {
        Fetched f{PAD_COORD, PAD_COORD, PAD_TIME, 0.0, INT_MAX};
        if (j < a.n) {
            f.x = a.x[j];
            f.y = a.y[j];
            f.t = a.t[j];
            const double sj = a.s[j];
            f.u = 1.0 / (sj * sj);
            f.g = a.g[j];
        }
        return f;
    };
    auto put = [&](int buf, const Fetched &f) {
        TileRecs &T = lt2[buf];
        T.x[tid] = f.x;
        T.y[tid] = f.y;
        T.t[tid] = f.t;
        T.u[tid] = f.u;
        T.q[tid] = f.u * a.qh;
        T.g[tid] = f.g;
    };
    const Rotation rot(li);

    for (int b = b_first; b < b_stop; ++b) {
        const int i0 = a.row_begin + b * TB;
        const int iend = (i0 + TB < a.row_end) ? i0 + TB : a.row_end;
        const double t_lo = a.t[i0], t_hi = a.t[iend - 1];
        // lanes past the block's end take a target far away: all of its terms are 0
        double xn[KT], yn[KT], tn[KT];
        int gn[KT];
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            const bool in = i < iend;
            xn[q] = in ? a.x[i] : PAD_COORD;
            yn[q] = in ? a.y[i] : PAD_COORD;
            tn[q] = in ? a.t[i] : PAD_TIME;
            gn[q] = in ? a.g[i] : INT_MAX;
        }
        double acc[KT][6];
#pragma unroll
        for (int q = 0; q < KT; ++q)
#pragma unroll
            for (int z = 0; z < 6; ++z)
                acc[q][z] = 0.0;

        const int k_strict = a.kstrict[b], k_end = a.kend[b];
        const int k0 = kg0;
        const int k1 = (kg1 < k_end) ? kg1 : k_end;

        if (k0 < k1)
            put(0, fetch(k0 * TS + tid));
        __syncthreads();

        for (int k = k0; k < k1; ++k) {
            const int buf = (k - k0) & 1;
            const bool more = (k + 1 < k1);
            Fetched next;
            if (more)
                next = fetch((k + 1) * TS + tid);

            const double first = a.tile[3 * k + 0], last = a.tile[3 * k + 1];
            const int cls = (last < t_lo) ? CAUSAL : ((first > t_hi) ? ANTI : MIXED);
            const bool cols = k < k_strict;  // strictly earlier block (so CAUSAL, whole tile)

            const char *lbase = reinterpret_cast<const char *>(&lt2[0]);
            const int tbase = buf * int(sizeof(TileRecs));
            struct Src {
                double x, y, t, u, q;
            };
            auto load = [&](int off) {
                const char *p = lbase + off;
                Src m;
                m.x = *reinterpret_cast<const double *>(p + offsetof(TileRecs, x));
                m.y = *reinterpret_cast<const double *>(p + offsetof(TileRecs, y));
                m.t = *reinterpret_cast<const double *>(p + offsetof(TileRecs, t));
                m.u = *reinterpret_cast<const double *>(p + offsetof(TileRecs, u));
                m.q = *reinterpret_cast<const double *>(p + offsetof(TileRecs, q));
                return m;
            };
            // One source for the lane's targets: background (BG, masked by tie group with
            // MASK; its column sums go to c0..c2) and triggering terms (TRIG, masked likewise).
            // The triggering exponent's spatial part t1 = u_m d2 qh serves the sum G1 too
            // (rescaled at the end).
            auto pair = [&](const Src &m, int gm, auto what, double &c0, double &c1, double &c2) {
                constexpr bool TRIG = (decltype(what)::value & 1) != 0, MASK = (decltype(what)::value & 2) != 0;
#pragma unroll
                for (int q = 0; q < KT; ++q) {
                    const double dx = xn[q] - m.x, dy = yn[q] - m.y, dt = tn[q] - m.t;
                    const double d2 = fma(dy, dy, dx * dx);
                    const double dt2 = dt * dt;
                    double bb = exp2_nonpos(-fma(a.at, dt2, a.ax * d2), ltab);
                    if (MASK)
                        bb = (gm != gn[q]) ? bb : 0.0;
                    acc[q][0] += bb;
                    c0 += bb;
                    if (GRAD) {
                        acc[q][1] = fma(bb, d2, acc[q][1]);
                        acc[q][2] = fma(bb, dt2, acc[q][2]);
                        c1 = fma(bb, d2, c1);
                        c2 = fma(bb, dt2, c2);
                    }
                    if (TRIG) {
                        const double t1 = m.q * d2;
                        double e = m.u * exp2_nonpos(-fma(a.omega, dt, t1), ltab);
                        if (MASK)
                            e = (gm < gn[q]) ? e : 0.0;
                        acc[q][3] += e;
                        if (GRAD) {
                            acc[q][4] = fma(e, t1, acc[q][4]);
                            acc[q][5] = fma(e, dt, acc[q][5]);
                        }
                    }
                }
            };
            auto pin_sums = [&]() {
#pragma unroll
                for (int q = 0; q < KT; ++q) {
                    if (GRAD)
                        pin(acc[q]);
                    else
                        asm volatile("" : "+v"(acc[q][0]), "+v"(acc[q][3]));
                }
                step_end();
            };
            using Trig = std::integral_constant<int, 1>;
            using Masked = std::integral_constant<int, 3>;
            using Anti = std::integral_constant<int, 0>;

            if (cols) {
                // 16-lane rotation: lane i takes source m0 + ((i + j) mod 16) at step j
                for (int m0 = mlo; m0 < mhi; m0 += 16) {
                    double e0 = 0.0, e1 = 0.0, e2 = 0.0;
                    auto half = [&](auto h) {
                        constexpr int HALF = decltype(h)::value;
                        const int base = tbase + m0 * 8;
                        Src m = load(rot.at(0, 64 * HALF, base));
#pragma unroll
                        for (int j = 0; j < GS; ++j) {
                            Src nx = m;
                            if (j + 1 < GS)
                                nx = load(rot.at(j + 1, 64 * HALF, base));
                            double c0 = -0.0, c1 = -0.0, c2 = -0.0;  // -0: first addition folds away
                            pair(m, 0, Trig{}, c0, c1, c2);
                            e0 = row_rotate_f64(e0) + c0;
                            if (GRAD) {
                                e1 = row_rotate_f64(e1) + c1;
                                e2 = row_rotate_f64(e2) + c2;
                            }
                            m = nx;
                            pin_sums();
                        }
                    };
                    half(std::integral_constant<int, 0>{});
                    half(std::integral_constant<int, 1>{});
                    // lane i of each row holds the row's sums of source m0 + ((i + 15) mod 16);
                    // row z of lanes ends with plane z
                    const double w = GRAD ? sum_rows4(e0, e1, e2, e2) : sum_rows_f64(e0);
                    if ((lane >> 4) < CP)
                        lcol[lane >> 4][wave][m0 + ((li + 15) & 15)] = w;
                }
            } else {
                const int mend = (k * TS + mhi <= a.n) ? mhi : a.n - k * TS;
                double c0 = -0.0, c1 = -0.0, c2 = -0.0;  // column sums unused
                const int *lg = lt2[buf].g;
                if (cls == CAUSAL) {
                    for (int m = mlo; m < mend; ++m)
                        pair(load(tbase + m * 8), 0, Trig{}, c0, c1, c2);
                } else if (cls == ANTI) {
                    for (int m = mlo; m < mend; ++m)
                        pair(load(tbase + m * 8), 0, Anti{}, c0, c1, c2);
                } else if (!(first == last && t_lo == t_hi && first == t_lo)) {  // one time for all: no terms
                    for (int m = mlo; m < mend; ++m)
                        pair(load(tbase + m * 8), lg[m], Masked{}, c0, c1, c2);
                }
            }

            if (more)
                put(buf ^ 1, next);
            __syncthreads();
            if (cols) {
                // owner lane of source tid: the four waves' sums in a fixed order
                const int j = k * TS + tid - jb;
                if (own) {
#pragma unroll
                    for (int z = 0; z < CP; ++z) {
                        double s = 0.0;
#pragma unroll
                        for (int w = 0; w < NW; ++w)
                            s += lcol[z][w][tid];
                        pc[z * cstride + j] += s;
                    }
                }
                __syncthreads();  // lcol is written again by the next tile's columns
            }
        }

        double *out = a.srow + int64_t(slot) * (GRAD ? 6 : 2) * stride;
#pragma unroll
        for (int q = 0; q < KT; ++q) {
            const int i = i0 + tid + q * WG;
            if (i >= iend)
                continue;
            const int rr = i - a.row_begin - rb0;
            out[0 * stride + rr] = acc[q][0];
            out[(GRAD ? 3 : 1) * stride + rr] = acc[q][3];
            if (GRAD) {
                out[1 * stride + rr] = acc[q][1];
                out[2 * stride + rr] = acc[q][2];
                out[4 * stride + rr] = acc[q][4] * a.out_g1;
                out[5 * stride + rr] = acc[q][5];
            }
        }
    }
}

constexpr int ROW_VALUES = 7;
struct Fin {
    const double *t, *x, *y, *s;   // raw events (the rescue sweep reads them)
    const int *g;                  // tie-group ids
    const int *status;             // [0] flags
    int *rescue_count, *ticket;
    int *rescue;                   // rescue list of row offsets
    double *rowvals;               // [row][7] l_n and gradient terms: of rescued rows, and sums of the others
    uint64_t *masks;               // the rescued rows among each 64
    double *lam_out, *comp_out;
    int64_t n, row_begin, rows;
    double mu, tau_x, tau_t, xi, h0, omega, c_b, c_g;
    double ax, at, qh;             // 1/(2 tau_x^2), 1/(2 tau_t^2), 1/(2 h0^2)
    double rescue_lambda;          // FP32 rows with lambda below this are recomputed (0: never)
    int uniform;                   // spatially uniform background: no tau_x dependence
};

__device__ inline double std_normal_cdf(double z) { return 0.5 * erfc(-z * 0.70710678118654752440); }
__device__ inline double std_normal_pdf(double z) { return 0.39894228040143267794 * exp(-0.5 * z * z); }

// From the six pair sums of row i (natural units): l_n, its six gradient
// terms, lambda_n and Lambda_n, all FP64.
template <bool GRAD>
__device__ void row_terms(const Fin &f, const double S[6], double ti, double tN, double v[7], double &lam,
                          double &comp)
{
    const double B = f.c_b * S[0];
    const double T = f.c_g * S[3];
    lam = f.mu * B + f.xi * T;
    const bool floored = !(lam >= LAMBDA_FLOOR);
    const double av = tN - ti;
    const double bg = std_normal_cdf(av / f.tau_t) - std_normal_cdf(-ti / f.tau_t);
    const double ea = exp(-f.omega * av);
    comp = f.mu * bg + f.xi * (1.0 - ea);
    v[0] = log(floored ? LAMBDA_FLOOR : lam) - comp;
    if (GRAD) {
        const double tx = f.tau_x, tt = f.tau_t, h0 = f.h0, om = f.omega;
        double dl[6] = {0, 0, 0, 0, 0, 0};
        if (!floored) {
            const double il = 1.0 / lam;
            dl[0] = B * il;
            dl[1] = f.uniform ? 0.0 : f.mu * f.c_b * (S[1] / (tx * tx * tx) - 2.0 * S[0] / tx) * il;
            dl[2] = f.mu * f.c_b * (S[2] / (tt * tt * tt) - S[0] / tt) * il;
            dl[3] = T * il;
            dl[4] = f.xi * f.c_g * (S[4] / (h0 * h0 * h0) - 2.0 * S[3] / h0) * il;
            dl[5] = f.xi * f.c_g * (S[3] / om - S[5]) * il;
        }
        const double dcomp_taut = -(f.mu / (tt * tt)) * (av * std_normal_pdf(av / tt) + ti * std_normal_pdf(ti / tt));
        v[1] = dl[0] - bg;
        v[2] = dl[1];
        v[3] = dl[2] - dcomp_taut;
        v[4] = dl[3] - (1.0 - ea);
        v[5] = dl[4];
        v[6] = dl[5] - f.xi * av * ea;
    }
}

// Fold of one pass: adds the slots of the pass's cells to each row's FP64
// accumulators, cell by cell in their launch order, so that the sums (and so
// the results) do not depend on where passes begin and end.  Row sums of row
// r come from the cells of its row group (column groups from the earliest
// up); in the symmetric sweep its column sums come from the cells of its
// column group (row groups from the latest down).  One thread per row and
// sum: a chain of additions whose loads are issued FOLD_AHEAD at a time, so
// that the fold streams the slots instead of waiting for each.
//   With FINAL (the last pass) the row's sums then meet in LDS and one thread
// per row does the FP64 finalize: lambda_n, the floored log, gradient terms,
// the compensator; the workgroup's 64 rows are added up.
struct FoldArgs {
    CellMap m;                // m.cell0, m.ncells: the cells of this pass
    int rr, cg, ge, sym;
    int first;                // the first pass: the accumulators start at zero
    int nrow, ncol;           // sums to fold: row planes rowz[0..nrow), column planes colz[0..ncol)
    int rowz[6], colz[3];
    int64_t row_step, col_step;  // slot strides
    int64_t rows, rows_pad;
    const double *srow, *scol;
    double *acc_row, *acc_col;  // [row plane][rows_pad], [column plane][rows_pad]
};

constexpr int FOLD_ROWS = 64;
constexpr int FOLD_AHEAD = 16;

// v plus count values, the i-th from at(i), added in that order
template <typename At>
__device__ inline double add_in_order(double v, int count, At at)
{
    int i = 0;
    for (; i + FOLD_AHEAD <= count; i += FOLD_AHEAD) {
        double x[FOLD_AHEAD];
#pragma unroll
        for (int k = 0; k < FOLD_AHEAD; ++k)
            x[k] = at(i + k);
#pragma unroll
        for (int k = 0; k < FOLD_AHEAD; ++k)
            v += x[k];
    }
    if (i < count) {  // the rest, with loads clamped to the last cell
        double x[FOLD_AHEAD];
#pragma unroll
        for (int k = 0; k < FOLD_AHEAD; ++k)
            x[k] = at(i + k < count ? i + k : count - 1);
#pragma unroll
        for (int k = 0; k < FOLD_AHEAD; ++k)
            v += (i + k < count) ? x[k] : -0.0;
    }
    return v;
}

template <bool GRAD, bool FINAL>
__global__ __launch_bounds__(FOLD_ROWS * 9) void k_fold(FoldArgs a, Fin f)
{
    __shared__ int lstart[MAX_SYM_GROUPS], lhi[MAX_SYM_GROUPS], llo[MAX_SYM_GROUPS];
    __shared__ double lsum[FINAL ? 9 : 1][FOLD_ROWS];
    const CellMap &m = a.m;
    const int z = threadIdx.y, c0 = m.cell0;
    int c1 = c0 + m.ncells;
    if (a.sym) {
        const int total = *m.total;
        c1 = c1 < total ? c1 : total;
        if (!FINAL && c0 >= c1 && !a.first)
            return;
        for (int g = z * FOLD_ROWS + threadIdx.x; g < m.num_gr; g += FOLD_ROWS * (a.nrow + a.ncol)) {
            lstart[g] = m.rowstart[g];
            lhi[g] = m.gchi[g];
            llo[g] = m.gclo[g];
        }
        __syncthreads();
    }
    const int64_t r = int64_t(blockIdx.x) * FOLD_ROWS + threadIdx.x;
    const bool in = r < a.rows;
    if (in && z < a.nrow) {
        const int zi = a.rowz[z];
        double *acc = a.acc_row + zi * a.rows_pad + r;
        const int gr = int((r / TB) / a.rr);
        const int rs = a.sym ? lstart[gr] : (m.num_gr - 1 - gr) * m.num_gc;
        const int nc = a.sym ? lhi[gr] - llo[gr] + 1 : m.num_gc;
        const int lo = rs > c0 ? rs : c0, hi = (rs + nc < c1) ? rs + nc : c1;
        double v = a.first ? 0.0 : *acc;
        const int64_t step = a.row_step;
        const double *p = a.srow + int64_t(lo - c0) * step + int64_t(zi) * a.ge + (r - int64_t(gr) * a.rr * TB);
        v = add_in_order(v, hi - lo, [&](int i) { return p[i * step]; });
        if (FINAL)
            lsum[z][threadIdx.x] = v;
        else
            *acc = v;
    } else if (in) {
        const int zi = a.colz[z - a.nrow];
        double *acc = a.acc_col + zi * a.rows_pad + r;
        const int gc = int(r / a.cg);
        // row groups whose cells hold column group gc: gclo <= gc <= gchi, a range since both
        // are nondecreasing; then those of this pass (cell numbers decrease with the row group)
        auto count_while = [&](int lo, auto pred) {  // first g >= lo for which pred fails
            int hi = m.num_gr;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (pred(mid))
                    lo = mid + 1;
                else
                    hi = mid;
            }
            return lo;
        };
        int gmin = count_while(0, [&](int g) { return lhi[g] < gc; });
        int gend = count_while(gmin, [&](int g) { return llo[g] <= gc; });
        auto cell = [&](int g) { return lstart[g] + gc - llo[g]; };
        gmin = count_while(gmin, [&](int g) { return g < gend && cell(g) >= c1; });
        gend = count_while(gmin, [&](int g) { return g < gend && cell(g) >= c0; });
        double v = a.first ? 0.0 : *acc;
        const double *p = a.scol + int64_t(zi) * a.cg + (r - int64_t(gc) * a.cg);
        v = add_in_order(v, gend - gmin,
                         [&](int i) { return p[int64_t(cell(gend - 1 - i) - c0) * a.col_step]; });
        if (FINAL)
            lsum[z][threadIdx.x] = v;
        else
            *acc = v;
    }
    if (!FINAL)
        return;
    __syncthreads();
    if (z != 0)
        return;
    double S[6] = {0, 0, 0, 0, 0, 0};
    const int x = in ? threadIdx.x : 0;
    if (GRAD) {
#pragma unroll
        for (int k = 0; k < 6; ++k)
            S[k] = lsum[k][x];
        if (a.ncol)
#pragma unroll
            for (int k = 0; k < 3; ++k)
                S[k] += lsum[6 + k][x];
    } else {
        S[0] = lsum[0][x];
        S[3] = lsum[1][x];
        if (a.ncol)
            S[0] += lsum[2][x];
    }
    const int64_t i = f.row_begin + (in ? r : f.rows - 1);
    double v[7] = {0, 0, 0, 0, 0, 0, 0}, lam, comp;
    row_terms<GRAD>(f, S, f.t[i], f.t[f.n - 1], v, lam, comp);
    const bool rescued = in && lam < f.rescue_lambda;
    if (rescued) {
        const int slot = atomicAdd(f.rescue_count, 1);
        f.rescue[slot] = int(r);
    }
    // the other rows' sums go to the first of them (the rescue writes the others' values)
    const uint64_t mask = __ballot(rescued);
    constexpr int nv = GRAD ? 7 : 1;
#pragma unroll
    for (int k = 0; k < nv; ++k) {
        v[k] = in && !rescued ? v[k] : 0.0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            v[k] += __shfl_xor(v[k], o);
    }
    if (!rescued && int(threadIdx.x) == __builtin_ctzll(~mask))
#pragma unroll
        for (int k = 0; k < nv; ++k)
            f.rowvals[r * ROW_VALUES + k] = v[k];
    if (threadIdx.x == 0)
        f.masks[blockIdx.x] = mask;
    if (!in)
        return;
    // per-row outputs are NaN where the data checks failed
    const bool bad = (f.lam_out || f.comp_out) && f.status[0] != 0;
    if (f.lam_out)
        f.lam_out[r] = bad ? __builtin_nan("") : lam;
    if (f.comp_out)
        f.comp_out[r] = bad ? __builtin_nan("") : comp;
}

constexpr int REDUCE_WG = 1024;
constexpr int REDUCE_WAVES = REDUCE_WG / 64;

// The sum over each row of 16 lanes, in every lane
__device__ __forceinline__ double row_sum_f64(double v)
{
    v += dpp_mov_f64<DPP_ROW_ROR8>(v);
    v += dpp_mov_f64<DPP_ROW_ROR4>(v);
    v += dpp_mov_f64<DPP_ROW_ROR2>(v);
    v += dpp_mov_f64<DPP_ROW_ROR1>(v);
    return v;
}

// FP64 rescue: rows whose FP32 rate is underflow-limited are swept again
// with every pair in FP64 (lanes strided over sources), and their row values
// are replaced.  Workgroups stride over the rescue list, so the grid size is
// independent of its length.  A row is taken by a team of 1 to 16 waves, whichever gets through the list
// in the fewest steps of 64 sources per wave, two of them (a sum over lanes, the row's terms, with more than one wave
// two barriers) counted for each round of rows: of a small set many rows are in flight, a wave each; a
// single row of a large one takes a whole workgroup.  Calls (value only, FP32) with teams of 4 waves, of 16,
// and so: every row of 100 events 291, 446, 63 us, of 700 729, 1083, 124, of 2,000 932, 1238, 169;
// one row in twenty of 20,000 732, 420, 405.
//   True in the threads that have written a row.
template <bool GRAD>
__device__ bool rescue_rows(const Fin &f, int count)
{
    bool wrote = false;
    __shared__ double part[6][REDUCE_WAVES];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int team = 1;  // waves per row
    uint64_t least = UINT64_MAX;
#pragma unroll
    for (int k = 0; 1 << k <= REDUCE_WAVES; ++k) {
        const unsigned at_once = gridDim.x * (REDUCE_WAVES >> k);
        const uint64_t steps = uint64_t((unsigned(count) + at_once - 1) / at_once) * (((f.n + (64 << k) - 1) >> (6 + k)) + 2);
        if (steps < least) {
            least = steps;
            team = 1 << k;
        }
    }
    const int rows = REDUCE_WAVES / team, own = wave / team, sub = wave % team;
    for (int w0 = blockIdx.x * rows; w0 < count; w0 += gridDim.x * rows) {
        const bool in = w0 + own < count;
        const int64_t r = f.rescue[in ? w0 + own : w0];
        const int64_t i = f.row_begin + r;
        const double xn = f.x[i], yn = f.y[i], tn = f.t[i];
        const int gn = f.g[i];
        double S[6] = {0, 0, 0, 0, 0, 0};
        for (int64_t m = 64 * sub + lane; m < f.n; m += 64 * team) {
            const int gm = f.g[m];
            if (gm == gn)
                continue;
            const double dx = xn - f.x[m], dy = yn - f.y[m];
            const double d2 = dx * dx + dy * dy;
            const double dt = tn - f.t[m];
            const double b = exp(-(f.ax * d2 + f.at * dt * dt));
            S[0] += b;
            S[1] += b * d2;
            S[2] += b * dt * dt;
            if (gm < gn) {
                const double sm = f.s[m];
                const double um = 1.0 / (sm * sm);
                const double e = um * exp(-(um * f.qh * d2 + f.omega * dt));
                S[3] += e;
                S[4] += e * (um * d2);
                S[5] += e * dt;
            }
        }
#pragma unroll
        for (int z = 0; z < 6; ++z)
            S[z] = sum_rows_f64(row_sum_f64(S[z]));
        if (team > 1) {  // a lane per wave of the team
            if (lane == 0)
#pragma unroll
                for (int z = 0; z < 6; ++z)
                    part[z][wave] = S[z];
            __syncthreads();
#pragma unroll
            for (int z = 0; z < 6; ++z)
                S[z] = row_sum_f64((lane & 15) < team ? part[z][own * team + (lane & 15)] : 0.0);
            __syncthreads();
        }
        if (in && sub == 0 && lane == 0) {
            double v[7] = {0, 0, 0, 0, 0, 0, 0}, lam, comp;
            row_terms<GRAD>(f, S, tn, f.t[f.n - 1], v, lam, comp);
            const int nv = GRAD ? 7 : 1;
            for (int z = 0; z < nv; ++z)
                f.rowvals[r * ROW_VALUES + z] = v[z];
            if (f.lam_out && f.status[0] == 0)
                f.lam_out[r] = lam;
            wrote = true;
        }
    }
    return wrote;
}

// Rescue and the sums of all rows, in one launch: with no row to rescue (as a rule) the
// first workgroup adds up the fold's sums of 64 rows; otherwise every workgroup
// takes its rows of the list and the last one to finish adds up, rescued rows
// after the sum of their 64.  Bound by launches and latency: as three launches
// (rescue, sums of 256 rows, their sum) a call of 5,000 events took 48.2 instead of 45.9 us,
// one of 20,000 144.0 instead of 141.6.  A row's values lie together, so that the first
// workgroup's strided reads touch one line per group (by planes it took 25 us at 1e5 rows,
// now 9).
template <bool GRAD>
__global__ __launch_bounds__(REDUCE_WG) void k_finish_rows(Fin f, int sums, double *loglik, double *grad)
{
    constexpr int nv = GRAD ? 7 : 1;
    __shared__ double red[nv][REDUCE_WAVES];
    __shared__ int last;
    const int tid = threadIdx.x, count = *f.rescue_count, bad = f.status[0];
    if (count == 0) {
        if (blockIdx.x != 0 || !sums)
            return;
    } else {
        const bool wrote = rescue_rows<GRAD>(f, count);
        if (!sums)
            return;
        if (wrote)
            __threadfence();  // the thread's rows before the workgroup's ticket
        __syncthreads();
        if (tid == 0)
            last = atomicAdd(f.ticket, 1) == int(gridDim.x) - 1;
        __syncthreads();
        if (!last)
            return;
        __threadfence();  // the others' rows after theirs
    }
    double v[nv];
#pragma unroll
    for (int z = 0; z < nv; ++z)
        v[z] = 0.0;
    auto add = [&](int64_t r) {
#pragma unroll
        for (int z = 0; z < nv; ++z)
            v[z] += f.rowvals[r * ROW_VALUES + z];
    };
    const int64_t groups = (f.rows + FOLD_ROWS - 1) / FOLD_ROWS;
    for (int64_t g = tid; g < groups; g += REDUCE_WG) {
        uint64_t mask = count ? f.masks[g] : 0;
        if (~mask)
            add(g * FOLD_ROWS + __builtin_ctzll(~mask));
        for (; mask; mask &= mask - 1)
            add(g * FOLD_ROWS + __builtin_ctzll(mask));
    }
#pragma unroll
    for (int z = 0; z < nv; ++z) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1)
            v[z] += __shfl_xor(v[z], o);
        if ((tid & 63) == 0)
            red[z][tid >> 6] = v[z];
    }
    __syncthreads();
    if (tid < nv) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < REDUCE_WAVES; ++w)
            s += red[tid][w];
        const double out = bad ? __builtin_nan("") : s;
        if (tid == 0) {
            if (loglik)
                loglik[0] = out;
        } else if (grad) {
            grad[tid - 1] = out;
        }
    }
}

// ------------------------------------------------------------ host side

thread_local char g_errbuf[512];

// Per-call tuning and timing (hawkes_options; defaults when absent).
struct Tuning {
    int64_t row_wgs = DEFAULT_ROW_WGS;
    int sym_groups = -1;  // group count; 0: whole-set calls take the row sweep, -1: the default plan
    hipEvent_t t_start = nullptr, t_stop = nullptr;
};

int parse_options(const hawkes_options *o, Tuning &T)
{
    if (!o)
        return HAWKES_OK;
    if (o->row_workgroups != 0) {
        if (o->row_workgroups < 1 || o->row_workgroups > MAX_ROW_WGS) {
            set_error("row_workgroups %lld outside [1, %lld]", (long long)o->row_workgroups,
                      (long long)MAX_ROW_WGS);
            return HAWKES_EINVAL;
        }
        T.row_wgs = o->row_workgroups;
    }
    if (o->symmetric_groups != 0) {
        if (o->symmetric_groups < -1 || o->symmetric_groups > MAX_SYM_GROUPS) {
            set_error("symmetric_groups %d outside [-1, %d]", int(o->symmetric_groups), MAX_SYM_GROUPS);
            return HAWKES_EINVAL;
        }
        T.sym_groups = o->symmetric_groups < 0 ? 0 : int(o->symmetric_groups);
    }
    if (o->reserved != 0) {
        set_error("hawkes_options.reserved must be 0");
        return HAWKES_EINVAL;
    }
    if ((o->timing_start == nullptr) != (o->timing_stop == nullptr)) {
        set_error("timing_start and timing_stop must both be set or both be NULL");
        return HAWKES_EINVAL;
    }
    T.t_start = reinterpret_cast<hipEvent_t>(o->timing_start);
    T.t_stop = reinterpret_cast<hipEvent_t>(o->timing_stop);
    return HAWKES_OK;
}

int validate(const hawkes_events *ev, const hawkes_theta *th, int precision, int64_t rb, int64_t re, const void *ws,
             size_t ws_bytes, Layout *L)
{
    if (!ev || !th) {
        set_error("null events or theta");
        return HAWKES_EINVAL;
    }
    if (ev->n < 1 || ev->n > MAX_N) {
        set_error("n = %lld outside [1, %lld]", (long long)ev->n, (long long)MAX_N);
        return HAWKES_EINVAL;
    }
    if (!ev->t || !ev->x || !ev->y || !ev->s) {
        set_error("null event array");
        return HAWKES_EINVAL;
    }
    if (!(ev->area >= 0.0) || !std::isfinite(ev->area)) {
        set_error("background area %g is not finite and >= 0", ev->area);
        return HAWKES_EINVAL;
    }
    if (!valid_precision(precision)) {
        set_error("precision %d is not HAWKES_FP64, HAWKES_FP32 or HAWKES_FP32_SKIP", precision);
        return HAWKES_EINVAL;
    }
    const double p[6] = {th->mu, th->tau_x, th->tau_t, th->xi, th->h0, th->omega};
    for (int k = 0; k < 6; ++k)
        if (!(p[k] > 0.0) || !std::isfinite(p[k])) {
            set_error("theta component %d = %g is not finite and positive", k, p[k]);
            return HAWKES_EINVAL;
        }
    if (rb < 0 || re > ev->n || rb > re) {
        set_error("row range [%lld, %lld) not within [0, %lld]", (long long)rb, (long long)re, (long long)ev->n);
        return HAWKES_ERANGE;
    }
    *L = make_layout(ev->n, precision);
    if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255u) != 0 || ws_bytes < L->minimum) {
        set_error("workspace %p of %zu bytes; need at least %zu bytes (%zu recommended), 256-byte aligned", ws,
                  ws_bytes, L->minimum, L->total);
        return HAWKES_EWORKSPACE;
    }
    return HAWKES_OK;
}

int record_event(hipEvent_t ev, hipStream_t stream)
{
    const hipError_t e = hipEventRecord(ev, stream);
    return e == hipSuccess ? HAWKES_OK : hip_failure(e, "hipEventRecord");
}

template <typename T>
T *at(void *ws, size_t off)
{
    return reinterpret_cast<T *>(static_cast<char *>(ws) + off);
}

enum Mode { MODE_LOGLIK, MODE_GRAD, MODE_TERMS };

// The slots of a pass: `cap` cells' row sums, then their column sums.
struct Slots {
    double *row = nullptr, *col = nullptr;
    int64_t cap = 0;
};

// The work plan of a call (cells and their slots) and its workspace arrays.
struct Setup {
    Plan P;
    SymPlan SP;
    bool sym = false, uniform = false;
    int64_t n = 0, rb = 0, re = 0, rows = 0;
    int *status = nullptr, *g = nullptr, *kstrict = nullptr, *kend = nullptr;
    double *tile = nullptr, *acc_row = nullptr, *acc_col = nullptr;
    CellMap cells;
    int rr = 1, cg = TB, ge = TB;  // target blocks and sources per group; rows per row group
    int row_planes = 6, col_planes = 3;  // sums the call's sweep writes
    double *slots = nullptr;         // the slot region
    size_t slot_avail = 0;
    double *early_slots = nullptr;   // the same with the row values' and the rescue list's space before it
    size_t early_avail = 0;
    int64_t cells_ub = 0, passes = 0, last_cell0 = 0;
    Slots early, last;               // of the last pass and of those before it
};

int setup(const hawkes_events *ev, int64_t rb, int64_t re, void *ws, size_t ws_bytes, const Layout &L,
          const Tuning &T, Setup &S)
{
    S.n = ev->n;
    S.rb = rb;
    S.re = re;
    S.rows = re - rb;
    S.uniform = ev->area > 0.0;
    S.status = at<int>(ws, L.status);
    S.g = at<int>(ws, L.g);
    S.tile = at<double>(ws, L.tile);
    S.kstrict = at<int>(ws, L.kstrict);
    S.kend = at<int>(ws, L.kend);

    // the plan, and whether one cell's slot fits, before any work is enqueued
    S.P = make_plan(S.rows > 0 ? S.rows : 1, L.num_tiles, T.row_wgs);
    // the symmetric sweep covers the whole event set; a row range takes the row sweep
    S.sym = T.sym_groups != 0 && rb == 0 && re == S.n;
    if (S.sym)
        S.SP = (T.sym_groups < 0) ? default_sym_plan(S.n) : make_sym_plan(S.n, T.sym_groups);
    const size_t cell_bytes = S.sym ? sym_cell_bytes(S.SP) : row_cell_bytes();
    S.slot_avail = ws_bytes - L.slots;
    if (S.slot_avail < cell_bytes) {
        set_error("workspace of %zu bytes leaves %zu bytes of slots; one cell of this plan needs %zu", ws_bytes,
                  S.slot_avail, cell_bytes);
        return HAWKES_EWORKSPACE;
    }
    // cells: row groups x column groups (the symmetric plan), or target blocks x source chunks
    S.rr = S.sym ? S.SP.rr : 1;
    S.cg = S.sym ? S.SP.cg : int(S.P.chunk_tiles * TS);
    S.ge = S.rr * TB;
    S.cells.num_gr = S.sym ? S.SP.num_gr : int(S.P.num_tb);
    S.cells.num_gc = S.sym ? S.SP.num_gc : int(S.P.num_chunks);
    if (S.sym) {
        S.cells.rowstart = at<int>(ws, L.rowstart);
        S.cells.gchi = at<int>(ws, L.gchi);
        S.cells.gclo = at<int>(ws, L.gclo);
        S.cells.total = S.cells.rowstart + MAX_SYM_GROUPS;
    }
    S.cells_ub = int64_t(S.cells.num_gr) * S.cells.num_gc;
    S.acc_row = at<double>(ws, L.acc);
    S.acc_col = S.acc_row + 6 * S.P.rows_pad;
    S.slots = at<double>(ws, L.slots);
    S.early_slots = at<double>(ws, L.rowvals);
    S.early_avail = ws_bytes - L.rowvals;
    return HAWKES_OK;
}

// FP32 source staging scales: positions by the background's spatial scale
// (or by the triggering bandwidth h0 when the background is spatially
// uniform), times by the temporal one.
struct StageF32 {
    double sx, st, rr, omega;
};

StageF32 stage_scales(const hawkes_theta *th, bool uniform)
{
    StageF32 sc;
    const double tau_sp = uniform ? th->h0 : th->tau_x;
    sc.sx = std::sqrt(LOG2E / (2.0 * tau_sp * tau_sp));
    sc.st = std::sqrt(LOG2E / (2.0 * th->tau_t * th->tau_t));
    sc.rr = (tau_sp / th->h0) * (tau_sp / th->h0);
    sc.omega = th->omega;
    return sc;
}

// The skip mode's ranges: background terms more than skip_gap days apart are
// exactly zero (scaled time gap whose square exceeds SKIP_EXPONENT), and the
// triggering culling range follows from omega.  Over several vectors the
// largest gap and the smallest omega.
struct SkipRange {
    bool on = false;
    double skip_gap = HUGE_VAL, omega = 0.0;
};

SkipRange skip_range(const hawkes_theta *th, int num_theta, int precision)
{
    SkipRange r;
    double max_tau_t = 0.0, min_omega = HUGE_VAL;
    for (int z = 0; z < num_theta; ++z) {
        max_tau_t = std::fmax(max_tau_t, th[z].tau_t);
        min_omega = std::fmin(min_omega, th[z].omega);
    }
    r.omega = min_omega;
    if (precision == HAWKES_FP32_SKIP) {
        r.on = true;
        r.skip_gap = std::sqrt(SKIP_EXPONENT) / std::sqrt(LOG2E / (2.0 * max_tau_t * max_tau_t));
    }
    return r;
}

// lambda_n = mu c_b S0 + xi c_g G0
struct RateScales {
    double c_b, c_g;
};

RateScales rate_scales(const hawkes_theta &th, double area)
{
    return {area > 0.0 ? 1.0 / (area * std::sqrt(2.0 * M_PI) * th.tau_t)
                       : 1.0 / (std::pow(2.0 * M_PI, 1.5) * th.tau_x * th.tau_x * th.tau_t),
            th.omega / (2.0 * M_PI * th.h0 * th.h0)};
}

// Events that bound a row's rate: more of them find larger bounds and so shorter ranges, at a cost of
// n times their number (a sweep costs n times the events in range, a constant share of n).
// Measured calls for 512 / 1024 / 2048 / 4096: gradient of 70,000 even events 783 / 787 / 814 / 867 us,
// of 100,000 in waves 1699 / 1646 / 1648 / 1703, of 300,000 14.08 / 13.52 / 13.29 / 13.33 ms, of 1e6
// 145.5 / 141.8 / 140.0 / 139.0 ms.
int64_t bound_sources(int64_t n)
{
    const int64_t want = ceil_div(n, 128 * BOUND_SOURCES) * BOUND_SOURCES;
    return want < MAX_BOUND_SOURCES ? want : MAX_BOUND_SOURCES;
}

BoundArgs bound_args(const hawkes_events *ev, const hawkes_theta *th, int num_theta, const Setup &S, const SkipRange &skip,
                     RateBound *out)
{
    BoundArgs b = {};
    b.t = ev->t;
    b.x = ev->x;
    b.y = ev->y;
    b.s = ev->s;
    b.n = S.n;
    b.out = out;
    b.groups = int(ceil_div(S.n, BOUND_ROWS));
    b.sources = int(bound_sources(S.n));
    // what is left of the gap where a rate of a single term's size makes up for the number of terms
    b.min_span = skip.skip_gap * std::sqrt(RATE_BITS / SKIP_EXPONENT);
    for (int z = 0; z < num_theta; ++z) {
        const hawkes_theta &h = th[z];
        const RateScales c = rate_scales(h, ev->area);
        b.ax[z] = S.uniform ? 0.0f : float(LOG2E / (2.0 * h.tau_x * h.tau_x));
        b.at[z] = float(LOG2E / (2.0 * h.tau_t * h.tau_t));
        b.qh[z] = float(LOG2E / (2.0 * h.h0 * h.h0));
        b.w[z] = float(h.omega * LOG2E);
        b.bg[z] = float(std::log2(h.mu * c.c_b));
        b.trig[z] = float(std::log2(h.xi * c.c_g));
        b.bg_unit[z] = float(std::log2(c.c_b * std::fmax(h.mu, 1.0)));
        b.trig_unit[z] = float(std::log2(c.c_g * std::fmax(h.xi, 1.0)));
    }
    return b;
}

// Stages the events (with the FP32 records of num_theta vectors) and plans the
// sweep's cells on the device.
int stage_and_plan(const hawkes_events *ev, const hawkes_theta *th, int num_theta, int precision, const Setup &S,
                   const Layout &L, void *ws, const SkipRange &skip, hipStream_t stream)
{
    int rc;
    StageArgs a = {};
    a.t = ev->t;
    a.x = ev->x;
    a.y = ev->y;
    a.s = ev->s;
    a.n = S.n;
    a.n_pad = L.n_pad;
    a.g = S.g;
    a.tile = S.tile;
    // the staging's per-workgroup results sit where the rescue masks will
    a.blocks = at<StageBlock>(ws, L.blocks);
    const unsigned blocks = unsigned(L.n_pad / 256);
    if (is_fp32(precision)) {
        a.xs = at<double>(ws, L.xs);
        a.ys = at<double>(ws, L.ys);
        a.tsd = at<double>(ws, L.tsd);
        a.r2 = at<float2>(ws, L.r2);
        a.v2 = at<float2>(ws, L.v2);
        a.u2 = at<float2>(ws, L.u2);
        a.dg = at<DeltaGroup>(ws, L.dg);
        a.theta_stride = L.n_pad;
        a.num_theta = num_theta;
        for (int z = 0; z < num_theta; ++z) {
            // r_m for each vector's own position scale; positions and times in the first's
            const StageF32 sc = stage_scales(th + z, S.uniform);
            if (z == 0) {
                a.sx = sc.sx;
                a.st = sc.st;
            }
            a.rr[z] = sc.rr;
            a.omega[z] = sc.omega;
        }
    }
    PlanArgs p = {};
    p.blocks = a.blocks;
    p.num_blocks = int(blocks);
    p.status = S.status;
    p.t = ev->t;
    p.tile = S.tile;
    p.n = S.n;
    p.num_tb = S.P.num_tb;
    p.row_begin = S.rb;
    p.row_end = S.re;
    p.num_tiles = int(L.num_tiles);
    p.sym = S.sym ? 1 : 0;
    p.trig_cull = skip.on ? 1 : 0;
    p.skip_gap = skip.skip_gap;
    p.omega = skip.omega;
    p.rr = S.rr;
    p.cg = S.cg;
    p.num_gr = S.cells.num_gr;
    p.kstrict = S.kstrict;
    p.kend = S.kend;
    p.gchi = at<int>(ws, L.gchi);
    p.gclo = at<int>(ws, L.gclo);
    p.rowstart = at<int>(ws, L.rowstart);
    p.total = p.rowstart + MAX_SYM_GROUPS;
    if (S.rows == 0)
        p.num_tb = 0;  // status words only
    const bool f32 = is_fp32(precision);
    if (S.n <= STAGE_PLAN_EVENTS) {
        if (f32)
            hipLaunchKernelGGL(k_stage_plan<true>, dim3(1), dim3(PLAN_WG), 0, stream, a, p);
        else
            hipLaunchKernelGGL(k_stage_plan<false>, dim3(1), dim3(PLAN_WG), 0, stream, a, p);
        return check_launch("stage_plan");
    }
    if (skip.on && S.rows > 0 && S.n > BOUND_EVENTS) {
        // scratch of the plan, in the accumulators that the first fold overwrites
        double *scratch = at<double>(ws, L.acc);
        p.far_trig = scratch;
        p.reach = scratch + L.num_tiles;
        const BoundArgs b = bound_args(ev, th, num_theta, S, skip,
                                       reinterpret_cast<RateBound *>(scratch + 2 * L.num_tiles));
        p.bounds = b.out;
        p.min_span = b.min_span;
        p.num_blocks = int(ceil_div(L.n_pad, 64 * BOUND_WAVES));
        const dim3 grid(unsigned(b.groups + p.num_blocks));
        if (num_theta == 1)
            hipLaunchKernelGGL(k_stage_bounds<1>, grid, dim3(64 * BOUND_WAVES), 0, stream, a, b);
        else
            hipLaunchKernelGGL(k_stage_bounds<MAX_FUSED_THETA>, grid, dim3(64 * BOUND_WAVES), 0, stream, a, b);
    } else if (f32)
        hipLaunchKernelGGL(k_stage<true>, dim3(blocks), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(k_stage<false>, dim3(blocks), dim3(256), 0, stream, a);
    if ((rc = check_launch("stage")) != HAWKES_OK)
        return rc;
    hipLaunchKernelGGL(k_plan, dim3(1), dim3(PLAN_WG), 0, stream, p);
    return check_launch("plan");
}

// Workgroups of `kernel` the device runs at once (0 if unknown).
int device_concurrency(const void *kernel)
{
    int dev = 0, cus = 0, per_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, WG, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return cus * per_cu;
}

// Pass plan: as many cells per pass as the slot region holds, rounded down to
// whole rounds of the workgroups the device runs at once (so that a pass ends
// without a ragged round of its own).  A slot holds only the sums the call's sweep
// writes (a third of all without the gradient).
//   Where that does not fill the device, the passes before the last also use the
// space of the row values and the rescue list (60 bytes per row), which the last
// pass's fold is the first to write.  At the minimum workspace the region holds one or two
// cells of the default plan, narrower than the square cell it is sized for; with those alone in a pass a
// gradient took 2.47, 19.8 and 96.3 ms at 2,000, 9,000 and 20,000 events (FP32), so it takes 0.51,
// 1.02 and 2.27 (0.05, 0.10 and 0.23 in the default workspace).
void plan_passes(Setup &S, const void *kernel, int row_planes, int col_planes)
{
    S.row_planes = row_planes;
    S.col_planes = S.sym ? col_planes : 0;
    const size_t cell = sizeof(double) * (size_t(row_planes) * S.ge + size_t(S.col_planes) * S.cg);
    auto slots = [&](double *p, size_t bytes, int64_t conc) {
        Slots s;
        s.cap = int64_t(bytes / cell);
        if (s.cap >= S.cells_ub)
            s.cap = S.cells_ub;
        else if (conc > 0 && s.cap > conc)
            s.cap -= s.cap % conc;
        s.row = p;
        s.col = p + s.cap * row_planes * S.ge;  // symmetric sweep: column slots after the row slots
        return s;
    };
    S.last = slots(S.slots, S.slot_avail, 0);
    if (S.last.cap == S.cells_ub) {
        S.early = S.last;
        S.passes = 1;
        S.last_cell0 = 0;
        return;
    }
    const int64_t conc = device_concurrency(kernel);
    S.last = slots(S.slots, S.slot_avail, conc);
    S.early = (S.last.cap < conc) ? slots(S.early_slots, S.early_avail, conc) : S.last;
    const int64_t early = ceil_div(S.cells_ub - S.last.cap, S.early.cap);
    S.passes = early + 1;
    S.last_cell0 = (early * S.early.cap < S.cells_ub) ? early * S.early.cap : S.cells_ub - S.last.cap;
}

// Which of the row and column planes of the slots a fold adds up.
struct FoldSums {
    int nrow = 0, ncol = 0;
    int rowz[6] = {0}, colz[3] = {0};
};

FoldArgs fold_args(const Setup &S, const Slots &slots, const FoldSums &z, int64_t cell0, int64_t ncells, bool first)
{
    FoldArgs fa = {};
    fa.m = S.cells;
    fa.m.cell0 = int(cell0);
    fa.m.ncells = int(ncells);
    fa.rr = S.rr;
    fa.cg = S.cg;
    fa.ge = S.ge;
    fa.sym = S.sym ? 1 : 0;
    fa.first = first ? 1 : 0;
    fa.nrow = z.nrow;
    fa.ncol = S.sym ? z.ncol : 0;
    for (int k = 0; k < 6; ++k)
        fa.rowz[k] = z.rowz[k];
    for (int k = 0; k < 3; ++k)
        fa.colz[k] = z.colz[k];
    fa.row_step = int64_t(S.row_planes) * S.ge;
    fa.col_step = int64_t(S.col_planes) * S.cg;
    fa.rows = S.rows;
    fa.rows_pad = S.P.rows_pad;
    fa.srow = slots.row;
    fa.scol = slots.col;
    fa.acc_row = S.acc_row;
    fa.acc_col = S.acc_col;
    return fa;
}

// Runs the sweep pass by pass: launches the pair kernel (launch(args, grid), args with the
// pass's cells and slots) and folds its slots (the sums `all`).  The last pass's fold
// is left to the caller, which runs it with the finalize (last_fold).
template <typename Args, typename Launch>
int sweep_passes(const Setup &S, const Tuning &T, const FoldSums &all, hipStream_t stream, Args a, Launch launch)
{
    int rc;
    if (T.t_start && (rc = record_event(T.t_start, stream)) != HAWKES_OK)
        return rc;
    for (int64_t p = 0; p < S.passes; ++p) {
        const bool last = (p + 1 == S.passes);
        const Slots &slots = last ? S.last : S.early;
        const int64_t cell0 = last ? S.last_cell0 : p * S.early.cap;
        const int64_t end = last ? S.cells_ub : (p + 2 == S.passes ? S.last_cell0 : cell0 + S.early.cap);
        a.cells.cell0 = int(cell0);
        a.cells.ncells = int(end - cell0);
        a.srow = slots.row;
        a.scol = slots.col;
        launch(a, dim3(unsigned(end - cell0)));
        if ((rc = check_launch("pair sweep")) != HAWKES_OK)
            return rc;
        if (last)
            break;
        const FoldArgs fa = fold_args(S, slots, all, cell0, end - cell0, p == 0);
        hipLaunchKernelGGL((k_fold<false, false>), dim3(unsigned(ceil_div(S.rows, FOLD_ROWS))),
                           dim3(FOLD_ROWS, unsigned(fa.nrow + fa.ncol)), 0, stream, fa, Fin{});
        if ((rc = check_launch("fold")) != HAWKES_OK)
            return rc;
    }
    return HAWKES_OK;
}

// The fold of the last pass.
FoldArgs last_fold(const Setup &S, const FoldSums &z)
{
    return fold_args(S, S.last, z, S.last_cell0, S.cells_ub - S.last_cell0, S.passes == 1);
}

// The sweep's cell fields shared by the pair kernels.
template <typename A>
void fill_grid(A &a, const Setup &S, const Layout &L)
{
    a.tile = S.tile;
    a.kstrict = S.kstrict;
    a.kend = S.kend;
    a.cells = S.cells;
    a.ge = S.ge;
    a.row_begin = int(S.rb);
    a.row_end = int(S.re);
    a.rows_pad = int(S.P.rows_pad);
    a.num_tiles = int(L.num_tiles);
    a.num_tb = int(S.P.num_tb);
    a.rr = S.rr;
    a.cg = S.cg;
    a.sym = S.sym ? 1 : 0;
}

Fin make_fin(const hawkes_events *ev, const hawkes_theta *th, int precision, const Setup &S, const Layout &L,
             void *ws, double *d_lam, double *d_comp)
{
    const double tau_x = th->tau_x, tau_t = th->tau_t, h0 = th->h0, omega = th->omega;
    Fin f;
    f.t = ev->t;
    f.x = ev->x;
    f.y = ev->y;
    f.s = ev->s;
    f.g = S.g;
    f.status = S.status;
    f.rescue_count = S.status + STATUS_RESCUE;
    f.ticket = S.status + STATUS_TICKET;
    f.rescue = at<int>(ws, L.rescue);
    f.rowvals = at<double>(ws, L.rowvals);
    f.masks = at<uint64_t>(ws, L.blocks);
    f.lam_out = d_lam;
    f.comp_out = d_comp;
    f.n = S.n;
    f.row_begin = S.rb;
    f.rows = S.rows;
    f.mu = th->mu;
    f.tau_x = tau_x;
    f.tau_t = tau_t;
    f.xi = th->xi;
    f.h0 = h0;
    f.omega = omega;
    f.uniform = S.uniform ? 1 : 0;
    const RateScales c = rate_scales(*th, ev->area);
    f.c_b = c.c_b;
    f.c_g = c.c_g;
    f.ax = S.uniform ? 0.0 : 1.0 / (2.0 * tau_x * tau_x);
    f.at = 1.0 / (2.0 * tau_t * tau_t);
    f.qh = 1.0 / (2.0 * h0 * h0);
    // Each FP32 pair term below 2^-126 may be lost to underflow; n of them
    // bound the loss by n 2^-126 (mu c_b + xi c_g).  Rows whose rate is not
    // 1/RESCUE_REL times larger than that are recomputed in FP64.
    f.rescue_lambda = is_fp32(precision)
                          ? double(S.n) * std::ldexp(1.0, -126) * (f.mu * f.c_b + f.xi * f.c_g) / RESCUE_REL
                          : 0.0;
    return f;
}

// After the last pair launch: its fold with the per-row finalize, FP64 rescue
// (FP32), and for the likelihoods the fixed-order reduction.  The second timing
// event (if any) follows the fold.
int finish(const Fin &f, const FoldArgs &fa, int precision, Mode mode, double *d_loglik, double *d_grad,
           hipEvent_t t_stop, hipStream_t stream)
{
    int rc;
    const bool grad = (mode == MODE_GRAD);
    const int64_t rows = f.rows;
    const dim3 grid(unsigned(ceil_div(rows, FOLD_ROWS))), block(FOLD_ROWS, unsigned(fa.nrow + fa.ncol));
    if (grad)
        hipLaunchKernelGGL((k_fold<true, true>), grid, block, 0, stream, fa, f);
    else
        hipLaunchKernelGGL((k_fold<false, true>), grid, block, 0, stream, fa, f);
    if ((rc = check_launch("finalize")) != HAWKES_OK)
        return rc;
    if (t_stop && (rc = record_event(t_stop, stream)) != HAWKES_OK)
        return rc;
    const bool f32 = is_fp32(precision);
    if (!f32 && mode == MODE_TERMS)
        return HAWKES_OK;  // the FP64 sweep has no rows to rescue
    const int64_t wgs = f32 ? ceil_div(rows, 256) : 1;
    const dim3 finish_grid(unsigned(wgs < 256 ? wgs : 256));
    const int sums = mode != MODE_TERMS;
    if (grad)
        hipLaunchKernelGGL(k_finish_rows<true>, finish_grid, dim3(REDUCE_WG), 0, stream, f, sums, d_loglik, d_grad);
    else
        hipLaunchKernelGGL(k_finish_rows<false>, finish_grid, dim3(REDUCE_WG), 0, stream, f, sums, d_loglik,
                           nullptr);
    return check_launch("finish_rows");
}

int run(const hawkes_events *ev, const hawkes_theta *th, int precision, int64_t rb, int64_t re, void *ws,
        size_t ws_bytes, const hawkes_options *opts, double *d_loglik, double *d_grad, double *d_lam,
        double *d_comp, Mode mode, void *stream_)
{
    Tuning T;
    int rc = parse_options(opts, T);
    if (rc != HAWKES_OK)
        return rc;
    Layout L;
    if ((rc = validate(ev, th, precision, rb, re, ws, ws_bytes, &L)) != HAWKES_OK)
        return rc;
    if (mode != MODE_TERMS && !d_loglik) {
        set_error("null loglik output");
        return HAWKES_EINVAL;
    }
    if (mode == MODE_GRAD && !d_grad) {
        set_error("null gradient output");
        return HAWKES_EINVAL;
    }
    hipStream_t stream = as_stream(stream_);
    const bool grad = (mode == MODE_GRAD);
    Setup S;
    if ((rc = setup(ev, rb, re, ws, ws_bytes, L, T, S)) != HAWKES_OK)
        return rc;
    const SkipRange skip = skip_range(th, 1, precision);
    if ((rc = stage_and_plan(ev, th, 1, precision, S, L, ws, skip, stream)) != HAWKES_OK)
        return rc;
    if (S.rows == 0) {
        if (mode != MODE_TERMS)
            hipLaunchKernelGGL(k_zero_outputs, dim3(1), dim3(64), 0, stream, d_loglik, grad ? d_grad : nullptr);
        return check_launch("zero_outputs");
    }
    const double h0 = th->h0, omega = th->omega;
    const bool uniform = S.uniform;
    // sums written by the sweeps: all of them with the gradient, S0 and G0 without
    FoldSums sums;
    if (grad)
        sums = FoldSums{6, 3, {0, 1, 2, 3, 4, 5}, {0, 1, 2}};
    else
        sums = FoldSums{2, 1, {0, 1}, {0}};

    if (is_fp32(precision)) {
        const StageF32 sc = stage_scales(th, uniform);
        const void *kfn = grad ? (uniform ? reinterpret_cast<const void *>(&k_pair_f32<true, true>)
                                          : reinterpret_cast<const void *>(&k_pair_f32<true, false>))
                               : (uniform ? reinterpret_cast<const void *>(&k_pair_f32<false, true>)
                                          : reinterpret_cast<const void *>(&k_pair_f32<false, false>));
        plan_passes(S, kfn, sums.nrow, sums.ncol);
        PairF32 a;
        fill_grid(a, S, L);
        a.xs = at<double>(ws, L.xs);
        a.ys = at<double>(ws, L.ys);
        a.tsd = at<double>(ws, L.tsd);
        a.t = ev->t;
        a.r2 = at<float2>(ws, L.r2);
        a.v2 = at<float2>(ws, L.v2);
        a.u2 = at<float2>(ws, L.u2);
        a.dg = at<DeltaGroup>(ws, L.dg);
        a.g = S.g;
        a.omega = omega;
        a.inv_st = 1.0 / sc.st;
        a.out_s1 = uniform ? 0.0 : 1.0 / (sc.sx * sc.sx);  // D = d^2 sx^2
        a.out_s2 = 1.0 / (sc.st * sc.st);        // dt' = dt st
        a.out_g1 = 2.0 * h0 * h0 / LOG2E;        // t1 = u d^2 log2(e) / (2 h0^2)
        a.w2 = omega * LOG2E / sc.st;
        a.out_exp = 1.0 / (1.0 + EXP2_MEAN_REL_ERR);
        a.trig_cull = skip.on ? 1 : 0;
        rc = sweep_passes(S, T, sums, stream, a, [&](const PairF32 &p, dim3 grid) {
            if (grad && uniform)
                hipLaunchKernelGGL((k_pair_f32<true, true>), grid, dim3(WG), 0, stream, p);
            else if (grad)
                hipLaunchKernelGGL((k_pair_f32<true, false>), grid, dim3(WG), 0, stream, p);
            else if (uniform)
                hipLaunchKernelGGL((k_pair_f32<false, true>), grid, dim3(WG), 0, stream, p);
            else
                hipLaunchKernelGGL((k_pair_f32<false, false>), grid, dim3(WG), 0, stream, p);
        });
    } else {
        const void *kfn = grad ? reinterpret_cast<const void *>(&k_pair_f64<true>)
                               : reinterpret_cast<const void *>(&k_pair_f64<false>);
        plan_passes(S, kfn, sums.nrow, sums.ncol);
        PairF64 a;
        fill_grid(a, S, L);
        a.t = ev->t;
        a.x = ev->x;
        a.y = ev->y;
        a.s = ev->s;
        a.g = S.g;
        a.n = int(S.n);
        // exponents in units of log2 (the sweep's exp2); uniform background: no spatial factor
        a.ax = uniform ? 0.0 : LOG2E / (2.0 * th->tau_x * th->tau_x);
        a.at = LOG2E / (2.0 * th->tau_t * th->tau_t);
        a.qh = LOG2E / (2.0 * h0 * h0);
        a.out_g1 = 2.0 * h0 * h0 / LOG2E;
        a.omega = omega * LOG2E;
        rc = sweep_passes(S, T, sums, stream, a, [&](const PairF64 &p, dim3 grid) {
            if (grad)
                hipLaunchKernelGGL(k_pair_f64<true>, grid, dim3(WG), 0, stream, p);
            else
                hipLaunchKernelGGL(k_pair_f64<false>, grid, dim3(WG), 0, stream, p);
        });
    }
    if (rc != HAWKES_OK)
        return rc;
    const Fin f = make_fin(ev, th, precision, S, L, ws, d_lam, d_comp);
    return finish(f, last_fold(S, sums), precision, mode, d_loglik, d_grad, T.t_stop, stream);
}

// Several parameter vectors on the same events and rows.  FP32: pairs of
// vectors share one forward-only sweep (k_pair_f32_batch), a vector left over
// takes the single sweep; FP64: one sweep per vector.
int run_batch(const hawkes_events *ev, const hawkes_theta *th, int64_t num_theta, int precision, int64_t rb,
              int64_t re, void *ws, size_t ws_bytes, const hawkes_options *opts, double *d_loglik, void *stream_)
{
    if (!th || num_theta < 1) {
        set_error("need at least one theta (got %lld, pointer %p)", (long long)num_theta, (const void *)th);
        return HAWKES_EINVAL;
    }
    if (!d_loglik) {
        set_error("null loglik output");
        return HAWKES_EINVAL;
    }
    Tuning T;
    int rc = parse_options(opts, T);
    if (rc != HAWKES_OK)
        return rc;
    Layout L;
    for (int64_t k = 0; k < num_theta; ++k)
        if ((rc = validate(ev, th + k, precision, rb, re, ws, ws_bytes, &L)) != HAWKES_OK)
            return rc;
    if (!is_fp32(precision) || num_theta == 1 || re == rb) {
        for (int64_t k = 0; k < num_theta; ++k)
            if ((rc = run(ev, th + k, precision, rb, re, ws, ws_bytes, opts, d_loglik + k, nullptr, nullptr,
                          nullptr, MODE_LOGLIK, stream_)) != HAWKES_OK)
                return rc;
        return HAWKES_OK;
    }
    hipStream_t stream = as_stream(stream_);
    Setup S;
    if ((rc = setup(ev, rb, re, ws, ws_bytes, L, T, S)) != HAWKES_OK)
        return rc;
    const void *kfn = S.uniform ? reinterpret_cast<const void *>(&k_pair_f32_batch<MAX_FUSED_THETA, true>)
                                : reinterpret_cast<const void *>(&k_pair_f32_batch<MAX_FUSED_THETA, false>);
    const FoldSums sums{2 * MAX_FUSED_THETA, MAX_FUSED_THETA, {0, 1, 2, 3}, {0, 1}};
    plan_passes(S, kfn, sums.nrow, sums.ncol);
    int64_t k = 0;
    for (; k + MAX_FUSED_THETA <= num_theta; k += MAX_FUSED_THETA) {
        const hawkes_theta *t0 = th + k;
        const SkipRange skip = skip_range(t0, MAX_FUSED_THETA, precision);
        if ((rc = stage_and_plan(ev, t0, MAX_FUSED_THETA, precision, S, L, ws, skip, stream)) != HAWKES_OK)
            return rc;
        const StageF32 sc0 = stage_scales(t0, S.uniform);
        PairBatchF32 a;
        fill_grid(a, S, L);
        a.xs = at<double>(ws, L.xs);
        a.ys = at<double>(ws, L.ys);
        a.tsd = at<double>(ws, L.tsd);
        a.t = ev->t;
        a.r2 = at<float2>(ws, L.r2);
        a.v2 = at<float2>(ws, L.v2);
        a.u2 = at<float2>(ws, L.u2);
        a.dg = at<DeltaGroup>(ws, L.dg);
        a.g = S.g;
        a.theta_stride = int(L.n_pad);
        a.out_exp = 1.0 / (1.0 + EXP2_MEAN_REL_ERR);
        const double tau_sp0 = S.uniform ? t0->h0 : t0->tau_x;
        for (int z = 0; z < MAX_FUSED_THETA; ++z) {
            const hawkes_theta *tz = t0 + z;
            const double tau_sp = S.uniform ? tz->h0 : tz->tau_x;
            a.cx[z] = (tau_sp0 / tau_sp) * (tau_sp0 / tau_sp);
            a.ct2[z] = (t0->tau_t / tz->tau_t) * (t0->tau_t / tz->tau_t);
            a.omega[z] = tz->omega;
            a.w2[z] = tz->omega * LOG2E / sc0.st;
        }
        a.trig_cull = skip.on ? 1 : 0;
        rc = sweep_passes(S, T, sums, stream, a, [&](const PairBatchF32 &p, dim3 grid) {
            if (S.uniform)
                hipLaunchKernelGGL((k_pair_f32_batch<MAX_FUSED_THETA, true>), grid, dim3(WG), 0, stream, p);
            else
                hipLaunchKernelGGL((k_pair_f32_batch<MAX_FUSED_THETA, false>), grid, dim3(WG), 0, stream, p);
        });
        if (rc != HAWKES_OK)
            return rc;
        for (int z = 0; z < MAX_FUSED_THETA; ++z) {
            // vector z's S0 and G0 are row planes z and 2 + z, its column sums plane z
            const FoldSums own{2, 1, {z, MAX_FUSED_THETA + z}, {z}};
            Fin f = make_fin(ev, t0 + z, precision, S, L, ws, nullptr, nullptr);
            f.rescue_count += z;
            f.ticket += z;
            if ((rc = finish(f, last_fold(S, own), precision, MODE_LOGLIK, d_loglik + k + z, nullptr,
                             z + 1 == MAX_FUSED_THETA ? T.t_stop : nullptr, stream)) != HAWKES_OK)
                return rc;
        }
    }
    for (; k < num_theta; ++k)
        if ((rc = run(ev, th + k, precision, rb, re, ws, ws_bytes, opts, d_loglik + k, nullptr, nullptr, nullptr,
                      MODE_LOGLIK, stream_)) != HAWKES_OK)
            return rc;
    return HAWKES_OK;
}

}  // namespace


void set_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_errbuf, sizeof(g_errbuf), fmt, ap);
    va_end(ap);
}

int hip_failure(hipError_t e, const char *what)
{
    set_error("%s: %s", what, hipGetErrorString(e));
    return HAWKES_EHIP;
}

int check_launch(const char *what)
{
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? HAWKES_OK : hip_failure(e, what);
}

}  // namespace hawkes

// ------------------------------------------------------------------ C ABI

using namespace hawkes;

extern "C" size_t hawkes_workspace_bytes(int64_t n, int precision)
{
    if (n < 1 || n > MAX_N || !valid_precision(precision))
        return 0;
    return make_layout(n, precision).total;
}

// ------------------------------------------------ the entry point that allocates nothing
//
// hawkes_loglik_grad_noalloc takes its workspace from a file-scope device
// array: every GPU the library runs on holds one copy of it at its own
// address until the process ends.  Host code never names the array as a
// pointer (that would be a host-side stand-in, not a device address): the
// device address is looked up once per device with hipGetSymbolAddress and
// kept.  Calls on one GPU share the array, so calls that overlap on one GPU
// race; every call writes what it reads afresh (status words and plan, staged
// records, and the accumulators in the first fold).

constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(64) << 20;
constexpr int NOALLOC_MAX_DEVICES = 64;

static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {

std::mutex g_scratch_mutex;
void *g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};

// The current device's address of `scratch` (looked up on the first call on that device).
int scratch_address(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return hip_failure(e, "hipGetDevice");
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) {
        set_error("device %d beyond the %d devices hawkes_loglik_grad_noalloc supports", dev, NOALLOC_MAX_DEVICES);
        return HAWKES_EINVAL;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess)
            return hip_failure(e, "hipGetSymbolAddress(scratch)");
        if (!p || (reinterpret_cast<uintptr_t>(p) & 255u) != 0) {
            set_error("scratch array of device %d at %p is not 256-byte aligned", dev, p);
            return HAWKES_EHIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return HAWKES_OK;
}

}  // namespace

extern "C" int hawkes_loglik_grad_noalloc(const hawkes_events *events, const hawkes_theta *theta, int precision,
                                          int64_t row_begin, int64_t row_end, double *d_loglik, double *d_grad,
                                          const hawkes_options *opts, void *stream)
{
    // host-side checks first (with a placeholder workspace address), so that invalid calls touch no device
    Layout L;
    int rc = validate(events, theta, precision, row_begin, row_end, reinterpret_cast<void *>(uintptr_t(256)),
                      SIZE_MAX, &L);
    if (rc != HAWKES_OK)
        return rc;
    if (L.minimum > NOALLOC_SCRATCH_BYTES) {
        set_error("n = %lld needs a workspace of at least %zu bytes at this precision; the static scratch of "
                  "hawkes_loglik_grad_noalloc holds %zu bytes",
                  (long long)events->n, L.minimum, NOALLOC_SCRATCH_BYTES);
        return HAWKES_EWORKSPACE;
    }
    void *ws = nullptr;
    if ((rc = scratch_address(&ws)) != HAWKES_OK)
        return rc;
    return run(events, theta, precision, row_begin, row_end, ws, NOALLOC_SCRATCH_BYTES, opts, d_loglik, d_grad,
               nullptr, nullptr, MODE_GRAD, stream);
}

extern "C" size_t hawkes_workspace_min_bytes(int64_t n, int precision)
{
    if (n < 1 || n > MAX_N || !valid_precision(precision))
        return 0;
    return make_layout(n, precision).minimum;
}

extern "C" int hawkes_loglik(const hawkes_events *events, const hawkes_theta *theta, int precision,
                             int64_t row_begin, int64_t row_end, void *ws, size_t ws_bytes, double *d_loglik,
                             const hawkes_options *opts, void *stream)
{
    return run(events, theta, precision, row_begin, row_end, ws, ws_bytes, opts, d_loglik, nullptr, nullptr,
               nullptr, MODE_LOGLIK, stream);
}

extern "C" int hawkes_loglik_grad(const hawkes_events *events, const hawkes_theta *theta, int precision,
                                  int64_t row_begin, int64_t row_end, void *ws, size_t ws_bytes, double *d_loglik,
                                  double *d_grad, const hawkes_options *opts, void *stream)
{
    return run(events, theta, precision, row_begin, row_end, ws, ws_bytes, opts, d_loglik, d_grad, nullptr,
               nullptr, MODE_GRAD, stream);
}

extern "C" int hawkes_event_terms(const hawkes_events *events, const hawkes_theta *theta, int precision,
                                  int64_t row_begin, int64_t row_end, void *ws, size_t ws_bytes, double *d_lambda,
                                  double *d_comp, const hawkes_options *opts, void *stream)
{
    return run(events, theta, precision, row_begin, row_end, ws, ws_bytes, opts, nullptr, nullptr, d_lambda,
               d_comp, MODE_TERMS, stream);
}

extern "C" int hawkes_loglik_batch(const hawkes_events *events, const hawkes_theta *thetas, int64_t num_theta,
                                   int precision, int64_t row_begin, int64_t row_end, void *ws, size_t ws_bytes,
                                   double *d_loglik, const hawkes_options *opts, void *stream)
{
    return run_batch(events, thetas, num_theta, precision, row_begin, row_end, ws, ws_bytes, opts, d_loglik,
                     stream);
}

extern "C" int hawkes_workspace_status(const void *ws, int *status, void *stream)
{
    if (!ws || !status) {
        set_error("null workspace or status pointer");
        return HAWKES_EINVAL;
    }
    int word = 0;
    hipError_t e = hipStreamSynchronize(as_stream(stream));
    if (e != hipSuccess)
        return hip_failure(e, "hipStreamSynchronize");
    e = hipMemcpy(&word, ws, sizeof(int), hipMemcpyDeviceToHost);
    if (e != hipSuccess)
        return hip_failure(e, "hipMemcpy(status)");
    *status = (word & STATUS_DATA) ? HAWKES_EDATA : ((word & STATUS_ORDER) ? HAWKES_EORDER : HAWKES_OK);
    return HAWKES_OK;
}

extern "C" const char *hawkes_strerror(int status)
{
    switch (status) {
    case HAWKES_OK: return "ok";
    case HAWKES_EINVAL: return "invalid argument";
    case HAWKES_ERANGE: return "row range out of bounds";
    case HAWKES_EWORKSPACE: return "workspace missing, misaligned or too small";
    case HAWKES_EHIP: return "HIP runtime error";
    case HAWKES_EORDER: return "event times are not sorted";
    case HAWKES_EDATA: return "non-finite event data or non-positive bandwidth scale";
    default: return "unknown status";
    }
}

extern "C" const char *hawkes_last_error(void) { return g_errbuf; }
