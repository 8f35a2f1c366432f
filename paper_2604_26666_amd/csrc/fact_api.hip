// C ABI of the library: argument validation, shape -> tile-configuration lookup, launches.
// Host code only; every step of the computation runs in the kernels of gemm_kernel.h and
// aux_kernels.hip.
#include "../../include/fact.h"
#include "launch.h"

#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

namespace fact {

static const ConfigDesc g_configs[] = {
#define FACT_CFG(id, bm, bn, wm, wn, bk, st) {id, bm, bn, wm, wn, bk, st, fact_launch_cfg##id},
#include "configs.def"
#undef FACT_CFG
};
static constexpr int kNumConfigs = (int)(sizeof(g_configs) / sizeof(g_configs[0]));

static constexpr int kNumCU = 256;
static constexpr int kLdsPerCU = 160 * 1024;
static constexpr int kMaxGridZ = 65535;
static constexpr size_t kStaticScratchBytes = (size_t)32 << 20;       // the array of fact_gemm_splitk_static

static thread_local char g_last_error[256] = "";

static int hip_fail(hipError_t e, const char *what)
{
    std::snprintf(g_last_error, sizeof g_last_error, "%s: %s", what, hipGetErrorString(e));
    return FACT_ERR_HIP;
}
int record_hip_failure(hipError_t e, const char *what) { return hip_fail(e, what); }    // for the other translation units

// ---- the per-shape table (filled by the on-device sweep) and the model behind it -----------

struct TableRow {
    int64_t batch, M, N, K;
    int trans_b, gated;
    int cfg, split, group_m;
};
static const TableRow g_table[] = {
#include "tile_table.inc"
    {0, 0, 0, 0, 0, 0, -1, 0, 0}   // sentinel
};

// Rows loaded at run time from a registry file (fact_registry_load): consulted before the
// compiled-in table, newest load first.  Readers and the loader share one mutex: a lookup is a
// short scan on the host and launches are asynchronous, so it is never held across GPU work.
static std::mutex g_registry_mutex;
static std::vector<TableRow> g_registry;

static bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

// Tail split hand-over: flags and the status word carry a launch-unique 64-bit value (a process-wide
// counter that starts at a clock-derived value), so a workspace never needs clearing and a stale
// word from another process or another use of the memory is not mistaken for one of ours.
static const unsigned long long g_tail_epoch_first =
    (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9E3779B97F4A7C15ull;
static std::atomic<unsigned long long> g_tail_epoch{g_tail_epoch_first};
static std::atomic<int> g_persistent{0};                  // fact_tune_persistent (off unless asked for: measured 0.5-3 % slower than ordinary launches)
static std::atomic<int> g_tail_budget{1 << 20};           // polls (about 0.3 us each) a collecting work-group waits: a third of a second

// Can the MFMA kernel take these operands at all?  (Dimensions only; pointer alignment is
// checked separately at launch.)
static bool fast_dims_ok(int64_t M, int64_t N, int64_t K, int trans_b)
{
    if (K % 8) return false;
    if (!trans_b && N % 8) return false;
    // (the kernel's rows and columns of a tile's edge, and k of a step ahead, are 32-bit: a wrapped edge would count as inside)
    if (M > INT32_MAX - 256 || N > INT32_MAX - 256 || K > INT32_MAX - 64) return false;
    return true;
}

static int wgs_per_cu(const ConfigDesc &c)
{
    int by_lds = kLdsPerCU / c.lds_bytes();
    // accumulators per lane + staging/fragment registers, out of 512 per lane at one wave per SIMD
    int acc = (c.bm / c.wm / 32) * (c.bn / c.wn / 32) * 16;
    int by_regs = 512 / (acc + 128);
    int occ = by_lds < by_regs ? by_lds : by_regs;
    return occ < 1 ? 1 : occ;
}

// Relative K-loop throughput of a compute unit running this tile, 256 x 256 = 1 (larger tiles reuse
// operands more).  Measured on a full chip at long K; the formula serves shapes of tile not listed.
static double tile_rate(const ConfigDesc &c)
{
    const int hi = c.bm > c.bn ? c.bm : c.bn, lo = c.bm > c.bn ? c.bn : c.bm;
    if (hi == 256 && lo == 256) return 1.0;
    if (hi == 256 && lo == 192) return 0.92;
    if (hi == 256 && lo == 128) return 0.85;
    if (hi == 192 && lo == 128) return 0.78;
    if (hi == 128 && lo == 128) return 0.74;
    if (hi == 64 && lo == 64) return 0.40;
    const double per_k = (double)(c.bm + c.bn) / ((double)c.bm * c.bn);   // operand bytes per MAC
    return (1.0 + 48.0 * 512.0 / 65536.0) / (1.0 + 48.0 * per_k);
}

// Work-groups of a persistent launch of `items` tiles (times batch entries) with K whole, or 0 when the
// launch is an ordinary one: every item fits at once, an 8-wave configuration (see the kernel), or
// switched off.  A multiple of 8, so a work-group stays on its XCD's part of the tile order.
static int persistent_grid(const ConfigDesc &c, int64_t items)
{
    if (c.wm * c.wn > 4 || !g_persistent.load(std::memory_order_relaxed)) return 0;
    const int64_t slots = (int64_t)kNumCU * wgs_per_cu(c);
    return items > slots && items <= INT32_MAX / 2 ? (int)slots : 0;
}

// A grid's threads are counted in 32 bits along x, and a larger count is cut without an error.
static bool grid_fits(const ConfigDesc &c, int64_t tiles) { return tiles <= (int64_t)UINT32_MAX / c.threads(); }
static int64_t tiles_of(const ConfigDesc &c, int64_t M, int64_t nout, bool gated)
{
    const int64_t bn_out = gated ? c.bn / 2 : c.bn;
    return (M + c.bm - 1) / c.bm * ((nout + bn_out - 1) / bn_out);
}
// Outputs that no configuration needs so many tiles for (at least 64 x 32 each, 512 threads at most): nothing to count.
static bool any_grid_fits(int64_t M, int64_t nout) { return M < 1 << 24 && nout < 1 << 24 && M * nout < (int64_t)1 << 33; }

struct Plan {
    int cfg = -1;      // -1: no tile configuration of the main kernel serves it (ragged or guarded kernel)
    int split = 1;
    int group_m = 4;
    bool loaded = false;   // from a registry file read at run time that says another thing than the compiled-in table
    // plan_one_round's choice, where it has one: it runs in the place of the above where the workspace of the call has room for its ranges.  (The call is
    // refused by the above's need alone: callers may have sized their workspaces by it.  Where that is nothing, a call without room for this one's ranges
    // is planned as one without a workspace.)
    int near_cfg = -1, near_split = 1;
    double near_us = 0.0;
    int most_ranges() const { return near_cfg >= 0 && near_split > split ? near_split : split; }
};

// Estimated microseconds of a launch, for shapes the registry does not list.  A 64-deep K step of a
// 256 x 256 tile takes 1.4 us on a busy chip; a tile costs 1.5 us + 1.5 us per 256 x 256 of area
// besides its K loop (first loads, epilogue); a partly filled last round runs its tiles up to a
// fifth faster (the chip is power-limited: fewer busy compute units, higher clock).  Checked against
// exhaustive timing of every configuration on 24 unlisted shapes: the choice costs 0.6 % on average
// and at most 8 % (the model it replaces, which counted the fixed cost in K steps and priced small
// tiles by a formula: 5.4 % and 30 %).
static constexpr int kModelConfigs = 16;         // the configurations it was fitted to; the others are plan_one_round's alone
static double model_time(const ConfigDesc &c, int64_t batch, int64_t M, int64_t nout, int64_t K, bool gated, int split)
{
    const int64_t bn_out = gated ? c.bn / 2 : c.bn;
    const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((nout + bn_out - 1) / bn_out) * batch * split;
    const int occ = wgs_per_cu(c);
    const int64_t slots = (int64_t)kNumCU * occ;
    const int64_t rounds = (tiles + slots - 1) / slots;
    const double area = (double)c.bm * c.bn / 65536.0;
    const double step_us = 1.40 * area / tile_rate(c);
    const int64_t ksteps = ((K + split - 1) / split + 63) / 64;
    const double tile_us = (double)occ * (double)ksteps * step_us + 1.5 + 1.5 * area;
    const double last = (double)(tiles - (rounds - 1) * slots) / (double)slots;     // how full the last round is
    return (double)(rounds - 1) * tile_us + tile_us * (1.0 - 0.2 * (1.0 - last));
}

// The plan of a launch of about one round of work-groups, K split or not, by the least estimated microseconds: what a step takes there is not the full
// chip's figure.  A compute unit's work-groups walk their K steps, each of them the longest of a latency (lat: an own one per tile), what the
// compute unit can pull of operands, and what the L2s deliver to all compute units together; then an epilogue; never faster than HBM
// delivers the operands; split K costs a launch and its planes.  Fitted to 62000 timed launches (1900 shapes of 65 to 8192 rows, 64 to 28672 columns,
// K of 64 to 131072, one to 256 ranges; mean error 9 %; on an independent sample 8 to 12 %, profiles/gemm_one_round_calls.csv).  Its choice against the best of all configurations and ranges, geometric mean over the
// shapes at which model_time chooses at most one round: K whole 1.5 %, with ranges 2.4 % ([N][K] 1.3 and 2.6; K of 8192 and more 2.4) where model_time's choice is
// 5.9, 8.0 and 15 % behind.  Beyond a round it is the other way round (4.8 and 1.6 %): epilogues run under other work-groups' steps there.
// Three sets: B as [K][N], as [N][K], and as [N][K] from 32 MB on, which a program with several such matrices finds in HBM (fitted to 28000 launches of 320
// shapes of 65 to 2048 rows whose weights were rotated out of the memory-side cache, plain and gated; mean error 5 %; the choice 1.2 % behind the best with K
// whole and 1.4 % with ranges; by the second set 2.7 and 5.8, by model_time 6.6 and 4.9).
struct RoundRates { double start, pull, chip, epilogue, memory, more, unaligned, reduce, planes; };
static constexpr RoundRates kRoundRates[3] = {{3.12, 117.2e3, 30.3e6, 10.4, 5.37e6, 1.157, 1.555, 5.3, 5.18e6}, {2.32, 95.3e3, 58.9e6, 10.4, 5.37e6, 1.157, 1.555, 5.3, 5.18e6},
                                              {1.0, 67.3e3, 48.1e6, 8.69, 5.31e6, 0.926, 1.622, 5.2, 6.56e6}};
struct StepLatency { int fit; bool choose; double lat[3]; };   // by configuration; fit: work-groups of a compute unit; us.  (What the ones not chosen from would add: 0.2 %.)
static constexpr StepLatency kStepLatency[] = {{1, true, {0.999, 0.975, 1.179}}, {1, false, {0.515, 0.530, 0.643}}, {1, true, {0.556, 0.542, 0.734}}, {2, false, {0.575, 0.566, 0.81}},
    {1, false, {0.505, 0.471, 0.641}}, {1, true, {0.510, 0.471, 0.742}}, {2, true, {0.194, 0.153, 0.065}}, {1, false, {0.358, 0.318, 0.506}}, {1, true, {0.338, 0.316, 0.513}},
    {1, false, {0.701, 0.670, 0.90}}, {1, false, {0.693, 0.687, 0.92}}, {1, false, {0.970, 0.927, 1.15}}, {1, false, {0.950, 0.920, 1.15}}, {1, true, {0.804, 0.804, 1.082}},
    {1, true, {0.450, 0.450, 0.629}}, {2, false, {0.645, 0.645, 0.90}}, {1, true, {0.249, 0.219, 0.263}}, {1, true, {0.275, 0.199, 0.341}}};
static_assert(sizeof(kStepLatency) / sizeof(kStepLatency[0]) == kNumConfigs, "a row for every configuration");
// How far the estimate has to be below the same estimate of model_time's plan, c0, to replace it (a factor; 0: never), by what the plans of 75000 random calls took, both timed
// (65 to 8192 rows, with and without a workspace, operands in the memory-side cache or rotated out of it; us, model_time's plan -> the other):
// * a tenth, where both split K or neither does: 1.08 to 1.25 times as fast in every class, 1 call in 100 of those that change more than 3 % slower;
// * 0.15 from 64 MB of operands on where B is [K][N] and the output at most 512 x 512 (45 calls that change between the two, at a tenth 1.08 times as fast in the cache and 0.93
//   out of it: 128 x 432 x 103104 35 -> 50; as [N][K] 36 calls 1.15 and 0.93, 424 x 112 x 71104 24.9 -> 21.0 and 28.0 -> 29.0; larger outputs, 68 calls, 1.15 and 1.21);
// * K whole in the place of ranges not from 64 MB on, where few work-groups would pull it all from HBM (94 x 11264 x 16728 [K][N] 97 -> 157, 8118 x 96 x 31360
//   107 -> 170).  Below, of 300 random calls and 47 feed-forward blocks that change between a tenth and 0.3: 0.3 with K of 4096 and more, outputs below 0.6 M elements and operands
//   of 8 MB and more (at a tenth 1.01 times as fast in the cache and 0.90 out of it; blocks 320 x 1024 x 4096 22.3 -> 23.9 and 27.3 -> 33.3), 0.2 from 32 MB on (at a tenth 1.02
//   and 0.94), and a tenth elsewhere: 1.10 and 1.03; blocks of 65 to 2048 tokens 1.08 and 1.00 (320 x 768 x 3072 19.1 -> 14.5 and 23.5 -> 17.6, 1237 x 1024 x 4096
//   44.2 -> 39.2 and 49.2 -> 48.0, 512 x 2048 x 5632 58.2 -> 52.6 and 59.4 -> 59.9);
// * ranges in the place of K whole, weights of 32 MB and more as [N][K], only from there on (621 x 3776 x 5568 35 -> 43 in the cache; beyond 1.15 times as fast out of
//   it and 1.06 in it).
// No tiles with ranges that are larger than c0's and than the output (130 x 72 x 16488 on 64 x 128 10.7 -> 12.7, 168 x 1704 x 30800 on 256 x 256 40 -> 53), and for [N][K] none
// of 256 x 192 and 256 x 256 whose rows are filled below 85 % (in the cache 0.9 times as fast; 797 x 592 x 29520 47 -> 58; above, 1.0 to 1.1).
static double clear_gain(const ConfigDesc &c, const ConfigDesc &c0, int64_t M, int64_t N, int64_t K, int trans_b, bool split, bool split0)
{
    const int64_t bytes = (M * K + N * K) * 2;
    const bool large = bytes >= (int64_t)64 << 20, weights = trans_b && N * K >= 1 << 24;      // (weights: the third set's)
    if (split && trans_b && ((c.bm > M && c.bm > c0.bm) || (c.bn > N && c.bn > c0.bn) || (c.bm * c.bn > 128 * 256 && 20 * M < 17 * ((M + c.bm - 1) / c.bm * c.bm)))) return 0.0;
    if (split0 && !split) return large ? 0.0 : K >= 4096 && M * N < 600000 && bytes >= 8000000 ? 0.7 : bytes >= (int64_t)32 << 20 ? 0.8 : 0.9;
    if (split && !split0) return large || !weights ? 0.9 : 0.0;
    return large && !trans_b && M * N <= 512 * 512 ? 0.85 : 0.9;
}

// ranges_asked: the ranges that the caller asks for (0: none asked for), at most kMaxGridZ: the launches counted here, of 4096 tiles at most, fit 32 bits.
// planes_held: the bytes of planes that this plan may choose ranges for.
static void plan_one_round(Plan &pl, int64_t M, int64_t N, int64_t nout, int64_t K, int trans_b, bool gated, bool allow_split, int ranges_asked, size_t planes_held)
{
    static constexpr int kRanges[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256};
    const int set = !trans_b ? 0 : N * K < 1 << 24 ? 1 : 2;
    const RoundRates &rates = kRoundRates[set];
    const int all_steps = ((int)K + 63) / 64;
    const double plane = (double)M * N * 8.0 / rates.planes, memory = rates.start + ((double)M * K + (double)N * K + (double)M * N) * 2.0 / rates.memory;
    struct Ranges { int asked, ksteps, count; double after; } ranges[sizeof(kRanges) / sizeof(kRanges[0])];
    auto in_ranges = [&](int asked) {
        Ranges r;
        r.asked = asked;
        r.ksteps = (all_steps + asked - 1) / asked;
        r.count = (all_steps + r.ksteps - 1) / r.ksteps;
        r.after = r.count > 1 ? rates.reduce + r.count * plane : 0.0;      // the reduction's launch, and its planes
        return r;
    };
    int choices = 0;
    for (const int s : kRanges) {
        if (s > 1 && (ranges_asked > 0 || !allow_split || all_steps < 4 * s || (size_t)s * M * N * sizeof(float) > planes_held)) break;
        ranges[choices++] = in_ranges(ranges_asked > 0 ? ranges_asked : s);
    }
    auto tiles_in = [&](const ConfigDesc &c) {
        const int bn_out = gated ? c.bn / 2 : c.bn;
        return ((int)M + c.bm - 1) / c.bm * (((int)nout + bn_out - 1) / bn_out);
    };
    auto estimate = [&](int cfg, int tiles, const Ranges &r) {
        const ConfigDesc &c = g_configs[cfg];
        const StepLatency &l = kStepLatency[cfg];
        const int slots = 256 * l.fit;
        const double area = rates.epilogue * (c.bm * c.bn) / 65536.0, lat = l.lat[set];
        const double bytes = 128.0 * ((M < c.bm ? M : c.bm) + (N < c.bn ? N : c.bn)) * (K % 64 ? rates.unaligned : 1.0);      // (rows that are no whole lines)
        const double own_us = bytes / rates.pull, all_us = bytes / rates.chip;
        auto step = [&](int sharing, int active) {
            const double own = sharing * own_us, all = active * all_us, most = own > all ? own : all;
            return most > lat ? most : lat;
        };
        int rem = tiles * r.count;
        double us = rates.start + 0.00555 * rem;
        if (rem > slots) {
            const int before = (rem - 1) / slots;
            rem -= before * slots;
            us += before * rates.more * (r.ksteps * step(l.fit, slots) + area * l.fit);
        }
        const int sharing = (rem + 255) / 256;
        us += r.ksteps * step(sharing, rem) + area * sharing;
        // (from HBM the two add up as much as they overlap)
        return (set == 2 ? std::sqrt(us * us + memory * memory) : us > memory ? us : memory) + r.after;
    };
    const Ranges before = in_ranges(ranges_asked > 0 ? ranges_asked : pl.split);
    const double before_us = estimate(pl.cfg, tiles_in(g_configs[pl.cfg]), before);
    for (int cfg = 0; cfg < kNumConfigs; ++cfg) {
        const ConfigDesc &c = g_configs[cfg];
        if (!kStepLatency[cfg].choose || !c.serves(trans_b)) continue;
        const int tiles = tiles_in(c);
        for (int i = 0; i < choices && (i == 0 || tiles * ranges[i].asked <= 512); ++i) {
            const double us = estimate(cfg, tiles, ranges[i]);
            if ((pl.near_cfg >= 0 && us >= pl.near_us) || us >= before_us * clear_gain(c, g_configs[pl.cfg], M, N, K, trans_b, ranges[i].asked > 1, before.asked > 1)) continue;
            pl.near_us = us;
            pl.near_cfg = cfg;
            pl.near_split = ranges[i].asked;
        }
    }
}

// (ranges_asked: as above, or kPlanned where the caller names a configuration or a tail split, so that only the plan's other parts are of use)
static constexpr int kPlanned = -1;
// planes_held: fact_gemm_splitk_static gives fact_gemm_splitk's results bit for bit, so where neither is asked for ranges both plan for what the static array
// holds (us, any number of planes -> 32 MiB of them, [N][K]: 962 x 5464 x 14040 203 -> 230, 1369 x 3656 x 13456 187 -> 215, 370 x 464 x 89168 73.3 -> 75.5,
// but 1067 x 6704 x 64504 1353 -> 1242).  The feed-forward block has no such twin and takes what it asks its caller for (1100 x 4096 x 14336 155 -> 137).
static Plan make_plan(int64_t batch, int64_t M, int64_t N, int64_t K, int trans_b, int act, bool allow_split, int ranges_asked = 0,
                      size_t planes_held = kStaticScratchBytes)
{
    Plan pl;
    const bool gated = act == FACT_ACT_SILU_GATE;
    if (!fast_dims_ok(M, N, K, trans_b)) return pl;
    auto matches = [&](const TableRow &r) {
        return r.batch == batch && r.M == M && r.N == N && r.K == K && r.trans_b == trans_b &&
               r.gated == (int)gated && (allow_split || (r.split >= 0 && r.split <= 1));
    };
    auto take = [&](const TableRow &r) {
        pl.cfg = r.cfg;
        pl.split = r.split == 0 ? 1 : r.split;             // negative: a tail split, which needs a workspace as well
        pl.group_m = r.group_m > 0 ? r.group_m : 4;
    };
    {
        std::lock_guard<std::mutex> lock(g_registry_mutex);
        for (const TableRow &r : g_registry)
            if (matches(r)) {
                take(r);
                // (the file that the table is generated from changes nothing when it is loaded)
                const TableRow *t = g_table;
                while (t->cfg >= 0 && !matches(*t)) ++t;
                pl.loaded = t->cfg < 0 || r.cfg != t->cfg || r.split != t->split || r.group_m != t->group_m;
                return pl;
            }
    }
    for (const TableRow *r = g_table; r->cfg >= 0; ++r)
        if (matches(*r)) { take(*r); return pl; }
    const int64_t nout = gated ? N / 2 : N;
    const bool all_fit = any_grid_fits(M, nout);
    double best = 0, whole = 0;
    int whole_cfg = -1;
    for (int i = 0; i < kModelConfigs; ++i) {
        const ConfigDesc &c = g_configs[i];
        if (gated && !c.gate_capable()) continue;
        if (!c.serves(trans_b) || (!all_fit && !grid_fits(c, tiles_of(c, M, nout, gated)))) continue;
        int max_split = 1;
        if (allow_split && batch == 1) {
            max_split = (int)(K / 1024);
            if (max_split > 256) max_split = 256;
            if (max_split < 1) max_split = 1;
        }
        for (int s = 1; s <= max_split; s *= 2) {
            double t = model_time(c, batch, M, nout, K, gated, s);
            if (s == 1 && (whole_cfg < 0 || t < whole)) { whole = t; whole_cfg = i; }
            if (s > 1) t += 4.0 + 2.0 * s * (double)M * N * 4.0 / 4.0e6;     // the reduction launch; partials written and read back at ~4 TB/s
            if (pl.cfg < 0 || t < best) { best = t; pl.cfg = i; pl.split = s; }
        }
    }
    // (Small ones for calls without K ranges are left to model_time: the choice is level, 0.5 and 0.7 % behind the best below 1 GFLOP, and takes a fraction of a microsecond
    // less; few rows have estimates of their own, few_rows_us.  A K of up to three steps is start and epilogue, which the estimate has the least of: 2368 x 2688 x 128
    // [K][N] 9.1 -> 10.7 us, 7715 x 560 x 184 8 % slower, others of [N][K] up to 3 % faster.)
    if (ranges_asked != kPlanned && batch == 1 && M > 64 && K >= 256 && all_fit && whole_cfg >= 0 && (allow_split || (double)M * N * K >= 0.5e9) &&
        tiles_of(g_configs[whole_cfg], M, nout, gated) <= kNumCU * wgs_per_cu(g_configs[whole_cfg]))
        plan_one_round(pl, M, N, nout, K, trans_b, gated, allow_split, ranges_asked, planes_held);
    pl.group_m = 4;
    return pl;
}

// ---- validation -----------------------------------------------------------------------------

struct Problem {
    int64_t batch, M, N, K;
    const void *A; int64_t lda, stride_a;
    const void *B; int64_t ldb, stride_b; int trans_b;
    const void *B_up;     // gated with separate weights, else nullptr
    void *C; int64_t ldc, stride_c;
    fact_epilogue ep;
    int store_stream = -1;    // of the call that this is a part of, -1: the call's own
};

static int validate(const Problem &q)
{
    if (!q.A || !q.B || !q.C) return FACT_ERR_NULL;
    if (q.batch <= 0 || q.M <= 0 || q.N <= 0 || q.K <= 0) return FACT_ERR_DIM;
    if (q.batch > kMaxGridZ) return FACT_ERR_DIM;
    if (q.trans_b != 0 && q.trans_b != 1) return FACT_ERR_LAYOUT;
    const int act = q.ep.act;
    if (act != FACT_ACT_NONE && act != FACT_ACT_GELU_TANH && act != FACT_ACT_SILU_GATE) return FACT_ERR_EPILOGUE;
    const bool gated = act == FACT_ACT_SILU_GATE;
    if (gated) {
        if (q.ep.bias) return FACT_ERR_EPILOGUE;
        if (q.N % 2) return FACT_ERR_EPILOGUE;
        if (!q.trans_b) return FACT_ERR_LAYOUT;
    }
    const int64_t nout = gated ? q.N / 2 : q.N;
    if (q.lda < q.K) return FACT_ERR_DIM;
    if (q.ldb < (q.trans_b ? q.K : q.N)) return FACT_ERR_DIM;
    if (q.ldc < nout) return FACT_ERR_DIM;
    if (q.ep.residual && q.ep.ldr < nout) return FACT_ERR_DIM;
    if (q.stride_a < 0 || q.stride_b < 0 || q.stride_c < 0 || q.ep.stride_r < 0) return FACT_ERR_DIM;
    if (q.batch > 1 && q.stride_c < (q.M - 1) * q.ldc + nout) return FACT_ERR_DIM;
    if (q.M > INT32_MAX || q.N > INT32_MAX || q.K > INT32_MAX) return FACT_ERR_DIM;
    const uintptr_t two = (uintptr_t)q.A | (uintptr_t)q.B | (uintptr_t)q.C | (uintptr_t)q.ep.bias |
                          (uintptr_t)q.ep.residual | (uintptr_t)q.B_up;
    if (two & 1u) return FACT_ERR_ALIGN;
    if (q.ep.out_f32 != 0 && q.ep.out_f32 != 1) return FACT_ERR_EPILOGUE;
    if (q.ep.f16 != 0 && q.ep.f16 != 1) return FACT_ERR_EPILOGUE;
    if (q.ep.out_f32 && ((uintptr_t)q.C & 3u)) return FACT_ERR_ALIGN;
    return FACT_OK;
}

static size_t splitk_ws_bytes(int64_t M, int64_t N, int split)
{
    return split > 1 ? (size_t)split * (size_t)M * (size_t)N * sizeof(float) : 0;
}

// Tail split: the tiles of the last, partly filled round are shared by g work-groups each.
struct TailPlan {
    int64_t first = 0;      // tiles computed whole
    int64_t rem = 0;        // tiles in the tail
    int g = 0;              // K ranges per tail tile (0: no tail split)
    // workspace: a status block (its first word: see fact_tail_timeouts), the fp32 partial tiles, one flag per partial
    static constexpr size_t kStatusBytes = 256;
    size_t bytes() const { return g > 1 ? kStatusBytes + (size_t)rem * (g - 1) * sizeof(float) * tile_floats + (size_t)rem * (g - 1) * 8 : 0; }
    size_t partials_offset() const { return kStatusBytes; }
    size_t flags_offset() const { return kStatusBytes + (size_t)rem * (g - 1) * sizeof(float) * tile_floats; }
    size_t tile_floats = 0;
};

static TailPlan tail_plan(const ConfigDesc &c, int64_t tiles, int64_t K, int g)
{
    TailPlan t;
    t.tile_floats = (size_t)c.bm * c.bn;
    const int64_t slots = (int64_t)kNumCU * wgs_per_cu(c);
    const int64_t ksteps = (K + 63) / 64;
    if (g < 2 || ksteps / g < 4) return t;            // too little K per range to be worth a hand-over
    if (!c.has_prefetch()) return t;                  // (no sink behind the ring: the collector has nowhere to pass its verdict)
    t.first = tiles / slots * slots;
    t.rem = tiles - t.first;
    if (t.rem == 0) { t.first = 0; return t; }
    t.g = g;
    return t;
}

// Column split: a launch whose last round of work-groups is partly filled runs as two, the columns of the full rounds
// on the plan's configuration and the rest on one that spreads them over the whole chip.
struct ColumnSplit {
    int64_t n1 = 0;        // output columns of the first launch (0: no split), a multiple of its tiles' width
    int cfg = -1;          // configuration of the second
};

// Where: the model has to see 6.5 % after 3 us for the second launch.  Measured on 30 shapes of 2 to 4 rounds (us, one
// launch -> two): 1024 x 50257 x 768 (3.08 rounds) 128.9 -> 102.4, 5018 x 6648 x 800 (2.03) 79.4 -> 70.8,
// 7268 x 2536 x 2552 (1.59) 118.4 -> 109.2, 5053 x 7608 x 6080 (2.34) 364.7 -> 346.0, 2048 x 28672 x 4096 (3.50) 368.5 ->
// 350.8; with less in it for the model the two are level or one launch is faster: 4980 x 8032 x 2936 (2.50) 221 -> 227,
// 5421 x 7864 x 1744 (2.66) 143 -> 146.  Configurations of which two work-groups share a compute unit fill a last round better
// than the model knows (8192 x 2304 x 768, 1.50 rounds: 31.2 -> 33.3) and are left alone; of those only the smallest tile
// takes a rest.
static ColumnSplit column_split(const Plan &pl, int64_t M, int64_t nout, int64_t K, int trans_b, bool gated)
{
    ColumnSplit sp;
    const ConfigDesc &c = g_configs[pl.cfg];
    if (wgs_per_cu(c) != 1) return sp;
    const int64_t bn_out = gated ? c.bn / 2 : c.bn;
    const int64_t tiles_m = (M + c.bm - 1) / c.bm, tiles = tiles_m * ((nout + bn_out - 1) / bn_out);
    const int64_t n1 = (tiles - 1) / kNumCU * kNumCU / tiles_m * bn_out;
    if (n1 <= 0 || n1 >= nout) return sp;
    const bool all_fit = any_grid_fits(M, nout);
    double rest = 0;
    for (int i = 0; i < kModelConfigs; ++i) {
        const ConfigDesc &d = g_configs[i];
        if ((gated && !d.gate_capable()) || !d.serves(trans_b) || (wgs_per_cu(d) > 1 && d.bm * d.bn > 64 * 64)) continue;
        if (!all_fit && !grid_fits(d, tiles_of(d, M, nout - n1, gated))) continue;
        const double t = model_time(d, 1, M, nout - n1, K, gated, 1);
        if (sp.cfg < 0 || t < rest) { rest = t; sp.cfg = i; }
    }
    if (sp.cfg >= 0 && model_time(c, 1, M, n1, K, gated, 1) + rest + 3.0 <= 0.935 * model_time(c, 1, M, nout, K, gated, 1)) sp.n1 = n1;
    return sp;
}

// Few rows against [N][K] weights: the skinny kernel, or the plan?  model_time prices full chips; with at most 64 rows a
// launch of the tile kernel is one or two rounds of work-groups that each wait for their loads: a K step is a load's latency
// or 60 GB/s per compute unit, the weights come at 5.0 TB/s (4.7 where their rows are no whole lines), and a split along K adds a launch of 5 us and its partial sums.
static double few_rows_us(const ConfigDesc &c, int64_t batch, int64_t M, int64_t N, int64_t nout, int64_t K, bool gated, int splits, bool whole_lines)
{
    const int64_t bn_out = gated ? c.bn / 2 : c.bn, tiles_n = (nout + bn_out - 1) / bn_out;
    const double tiles = (double)((M + c.bm - 1) / c.bm) * tiles_n * batch * splits;
    const int fit = wgs_per_cu(c);
    const double rounds = tiles > 256.0 * fit ? tiles / (256.0 * fit) : 1.0;
    const double sharing = tiles < 256.0 ? 1.0 : tiles / 256.0 < fit ? tiles / 256.0 : fit;
    const double bytes = 128.0 * ((M < c.bm ? M : c.bm) + (N < c.bn ? N : c.bn)), step = sharing * bytes / 60e3;
    const double latency = c.bm == 64 ? 0.2 : 0.5 * std::sqrt((double)c.bm * c.bn / 65536.0);
    const int64_t ksteps = ((K + splits - 1) / splits + 63) / 64;
    const double chain = 3.2 + 0.0086 * tiles + rounds * (double)ksteps * (step > latency ? step : latency);
    const double memory = 3.2 + (double)batch * K * 2.0 * (N + (double)(tiles_n < 8 ? tiles_n : 8) * M) / (whole_lines ? 5.0e6 : 4.7e6);
    return (chain > memory ? chain : memory) + (splits > 1 ? 5.0 + (double)M * N * 8.0 * splits / 1e7 : 0.0);
}

// The plan's time where the chip has few work-groups of it: model_time prices full chips.  Fitted to the same calls as
// small_us, of which those with more than 64 rows or B as [K][N] ran the tile kernel (mean error 13 and 6 %).
static double small_plan_us(const ConfigDesc &c, bool trans_b, int64_t batch, int64_t M, int64_t N, int64_t K, int splits)
{
    const int64_t tiles_n = (N + c.bn - 1) / c.bn;
    const double tiles = (double)((M + c.bm - 1) / c.bm) * tiles_n * batch * splits;
    const int fit = wgs_per_cu(c);
    const double rounds = tiles > 256.0 * fit ? tiles / (256.0 * fit) : 1.0;
    const double sharing = tiles < 256.0 ? 1.0 : tiles / 256.0 < fit ? tiles / 256.0 : fit;
    const double area = (double)c.bm * c.bn / 65536.0, latency = c.bm == 64 ? (trans_b ? 0.124 : 0.184) : 0.5 * std::sqrt(area);
    const double step = sharing * 128.0 * ((M < c.bm ? M : c.bm) + (N < c.bn ? N : c.bn)) / (trans_b ? 84.1e3 : 71.4e3);
    const int64_t ksteps = ((K + splits - 1) / splits + 63) / 64;
    const double start = trans_b ? 3.06 : 4.16;
    const double chain = start + 0.004 * tiles + rounds * ((trans_b ? 14.7 : 8.2) * area + (double)ksteps * (step > latency ? step : latency));
    const double memory = start + (double)batch * K * 2.0 * (N + (double)(tiles_n < 8 ? tiles_n : 8) * M) / 5.0e6;
    return (chain > memory ? chain : memory) + (splits > 1 ? 4.0 + (double)M * N * 8.0 * splits / 1e7 : 0.0);
}

// Which form of the skinny kernel runs in the plan's place: kFewRows, a tile of small_us, or kNoSkinny.
// Few rows where the skinny kernel's estimate (skinny_us) is below the plan's (few_rows_us).  Both were fitted to 1100 calls of 1 to 64 rows, 16 to
// 36000 columns, K of 64 to 131072 and batches up to 128, with and without a workspace, operands from HBM; the choice costs
// 0.4 % over the better kernel of every call on average; in 28 of them the one it takes is more than 3 % slower, by 25 % at most
// but for two (46 and 49 %).  Some of the calls (us, plan -> skinny; * the plan is kept):
//    M x N x K:  16 x 4096 x 14336  59.6 -> 25.6     16 x 768 x 3072  9.5 -> 6.3       64 x 3072 x 768  5.3 -> 4.4
//                16 x 16384 x 8192  62.6 -> 52.0     16 x 16384 x 256  5.4 -> 6.6 *    32 x 16384 x 1024  9.6 -> 11.2 *
//    with a workspace, so that the plan may split K:
//                16 x 64 x 8192  11.7 -> 10.3        16 x 64 x 32768  12.0 -> 34.9 *   64 x 64 x 131072  16.6 -> 315 *
//    without:    16 x 64 x 8192  23.7 -> 10.4        64 x 64 x 32768  134 -> 51        64 x 64 x 131072  559 -> 318
//    batches:    8 x (16 x 256 x 1024)  6.7 -> 4.1   128 x (32 x 64 x 4096)  24.8 -> 37.2 *   128 x (64 x 512 x 1024)  33.1 -> 75.4 *
// Small outputs (small_us) where the estimate is 8 % below the plan's (us, plan -> skinny; M x N x K): B as [K][N] 43 x 2736 x 80 5.3 -> 3.6, 1 x 32 x 3688
// 15.0 -> 5.7, 22 x 176 x 3920 16.0 -> 7.6, 120 x 112 x 6280 31.3 -> 13.3, 610 x 344 x 7272 36.3 -> 23.7; but 159 x 5840 x 928 12.2 -> 16.8; [N][K]
// 67 x 56 x 256 4.7 -> 3.3, 425 x 104 x 1352 7.2 -> 4.5, 180 x 1920 x 600 6.0 -> 5.1; but 572 x 1552 x 2128 14.8 -> 25.  Over the 650 calls with more than 64
// rows or B as [K][N] the choice is 1.29 and 1.50 times as fast as the plan alone, the better kernel of every call 1.34 and 1.55 times;
// 4 of them lose more than 3 %, 12 % at most.  The estimates of small outputs are of operands in the memory-side cache; cold ones (60 random calls each,
// caches filled with other data) are 1.62 and 1.33 times as fast as the plan, warm ones 1.66 and 1.28 times.
static constexpr int kNoSkinny = -2, kFewRows = -1;
// c, splits: model_time's plan.  plan_us: plan_one_round's estimate of the one that runs in its place, or 0.
static int skinny_choice(const GemmArgs &a, bool trans_b, int64_t batch, const ConfigDesc &c, int splits, double plan_us)
{
    const bool gated = a.act == FACT_ACT_SILU_GATE, few = skinny_takes(a, trans_b);
    const bool lines = ((uintptr_t)a.B & 127u) == 0 && a.ldb % 64 == 0 && (batch == 1 || a.stride_b % 64 == 0);
    int tile = -1;
    const double small = small_us(a, trans_b, batch, 0, &tile);
    // (A plan that splits K is quicker than its estimate, by what its reduction became, and a K as long as that longer here: with a workspace us, plan and
    // this kernel at their estimates' ratio: [N][K] 80 x 304 x 15168 13.1 / 13.8 at 0.86, 352 x 328 x 6848 13.2 / 14.7 at 0.90, but 280 x 120 x 7232 13.1 / 8.7 at
    // 0.77; [K][N] 256 x 64 x 8192 10.4 / 14.0 at 0.87, 160 x 64 x 7680 13.4 / 13.6 at 0.67, but 72 x 64 x 5888 11.7 / 10.3 at 0.62.)
    const double line = splits <= 1 ? 0.92 : trans_b ? 0.8 : 0.65;
    if (!few) {
        const bool taken = tile >= 0 && small < line * small_plan_us(c, trans_b, batch, a.M, a.N, a.K, splits);
        if (plan_us <= 0.0) return taken ? tile : kNoSkinny;
        // The plan is another one, priced by plan_one_round, and the small tiles of [N][K] by rates of the same measurements.  What was taken stays taken (us, small tile and
        // the plan with ranges that is estimated a fifth below it, from the cache: 0.76 times as fast as [K][N], 69 calls, 0.89 as [N][K], 239), with the tile that those rates
        // name where a compute unit has one work-group of it (770 calls 1.18 times as fast; with two 0.92).  Otherwise the small tiles run in the place of K whole below 1.1 of the
        // plan's estimate, and of ranges below 0.9 ([K][N] 0.83): 490 calls 1.28 times as fast as model_time's plan; not with rows of odd lengths from 4096 on (0.91: 464 x 224 x 5912
        // 12.5 -> 17.1), nor where many compute units have two (229 x 1224 x 3072, 312 work-groups, 12.4 -> 15.3; up to 288 1.28).
        int other = -1;
        const double other_us = small_us(a, trans_b, batch, taken ? 256 : 288, &other);
        if (taken) return trans_b && other >= 0 ? other : tile;
        if (other < 0 || (a.splits > 1 && trans_b && a.K % 64 && a.K >= 4096)) return kNoSkinny;
        return other_us < (a.splits <= 1 ? 1.1 : trans_b ? 0.9 : 0.83) * plan_us ? other : kNoSkinny;
    }
    const double rows = skinny_us(a, batch, lines), plan = few_rows_us(c, batch, a.M, a.N, gated ? a.N / 2 : a.N, a.K, gated, splits, lines);
    if (rows < plan || (splits <= 1 && tile >= 0 && small < 0.92 * plan)) return tile >= 0 && small < rows ? tile : kFewRows;
    return kNoSkinny;
}

// ---- the one launch path every entry point goes through ----------------------------------------

// The second GEMM of the feed-forward block: as many planes as its own workspace query asks for.
static Plan down_plan(int64_t T, int64_t d_model, int64_t d_ff) { return make_plan(1, T, d_model, d_ff, 1, FACT_ACT_NONE, true, 0, SIZE_MAX); }

// How a call runs, for fact_test_route: with one of these run() notes each launch in place of making it.
struct Route {
    static constexpr int kMax = 4;
    int launches = 0;
    int kind[kMax], cfg[kMax], streams[kMax];
    int64_t columns[kMax];           // contraction columns of the launch
    int add(int k, int c, int64_t n, int stream = 0) { if (launches < kMax) { kind[launches] = k; cfg[launches] = c; columns[launches] = n; streams[launches] = stream; } ++launches; return FACT_OK; }
};

static thread_local Route g_last_route;      // of the thread's last fact_test_route

static int run(const Problem &q, int cfg_id, int split, int group_m, bool allow_table_split,
               void *ws, size_t ws_bytes, hipStream_t stream, Route *route = nullptr, const Plan *given = nullptr)
{
    int rc = validate(q);
    if (rc != FACT_OK) return rc;
    if (split > kMaxGridZ) return FACT_ERR_UNSUPPORTED;
    const bool gated = q.ep.act == FACT_ACT_SILU_GATE;
    const int64_t nout = gated ? q.N / 2 : q.N;

    Plan pl = given ? *given : make_plan(q.batch, q.M, q.N, q.K, q.trans_b, q.ep.act, allow_table_split, cfg_id >= 0 || cfg_id == FACT_CONFIG_GUARDED || split < 0 ? kPlanned : split);
    double near_us = 0.0;
    int before_cfg = -1, before_split = 1;            // what plan_one_round's choice replaces
    if (pl.near_cfg >= 0) {
        auto has_room = [&](int ranges) { return ranges <= 1 || (ws && aligned16(ws) && ws_bytes >= splitk_ws_bytes(q.M, q.N, ranges)); };
        if (split == 0 && pl.split <= 1 && !has_room(pl.near_split)) pl = make_plan(q.batch, q.M, q.N, q.K, q.trans_b, q.ep.act, false);
        if (pl.near_cfg >= 0 && (split > 0 || (has_room(pl.split) && has_room(pl.near_split)))) {
            before_cfg = pl.cfg;
            before_split = split > 0 ? split : pl.split;
            pl.cfg = pl.near_cfg;
            pl.split = pl.near_split;
            near_us = q.trans_b && q.N * q.K >= 1 << 24 ? 0.0 : pl.near_us;      // (skinny_choice's lines for it are of warm operands)
        }
    }
    if (cfg_id == FACT_CONFIG_GUARDED) {              // the guarded kernel on request: the sweep's reference result
        if (split > 1 || split < 0 || q.ep.out_f32) return FACT_ERR_UNSUPPORTED;
        pl.cfg = -1; pl.split = 1;
    }
    if (cfg_id >= 0) {
        if (cfg_id >= kNumConfigs) return FACT_ERR_UNSUPPORTED;
        if (!fast_dims_ok(q.M, q.N, q.K, q.trans_b)) return FACT_ERR_UNSUPPORTED;
        if (gated && !g_configs[cfg_id].gate_capable()) return FACT_ERR_UNSUPPORTED;
        if (!g_configs[cfg_id].serves(q.trans_b)) return FACT_ERR_UNSUPPORTED;
        pl.cfg = cfg_id;
        if (split <= 0) pl.split = 1;
    }
    if (split > 0) pl.split = split;
    if (split < 0) pl.split = split;                  // forced tail split, -split ranges per tail tile
    if (group_m > 0) pl.group_m = group_m;
    int tail_g = 0;                                   // a negative split in a plan is a tail split
    if (pl.split < 0) { tail_g = -pl.split; pl.split = 1; }
    if (tail_g > 1 && q.batch != 1) { if (split < 0) return FACT_ERR_UNSUPPORTED; tail_g = 0; }
    if (pl.split > 1 && q.batch != 1) return FACT_ERR_UNSUPPORTED;

    // operands the MFMA kernel reads with 16-byte loads
    // (leading dimensions are bounded so that per-lane byte offsets inside one tile panel fit 31 bits)
    const bool ptr_ok = aligned16(q.A) && aligned16(q.B) && (!q.B_up || aligned16(q.B_up)) &&
                        q.lda % 8 == 0 && q.ldb % 8 == 0 && q.stride_a % 8 == 0 && q.stride_b % 8 == 0 &&
                        q.lda <= (1 << 21) && q.ldb <= (1 << 21);
    if (pl.cfg >= 0 && !ptr_ok) {
        if (cfg_id >= 0) return FACT_ERR_UNSUPPORTED;
        pl.cfg = -1;
    }
    if (pl.cfg < 0) pl.split = 1;     // the fallback never splits
    // fp32 output: with K whole the main kernel's epilogue writes it, unrounded; with K split the
    // reduction pass does (no batch then, as for any split).  No tail split, no fallback kernel.
    bool out_f32 = q.ep.out_f32 != 0, c_f32 = false;
    if (out_f32) {
        if (pl.cfg < 0) return FACT_ERR_UNSUPPORTED;
        tail_g = 0;
        if (pl.split < 1) pl.split = 1;
        if (pl.split == 1) { c_f32 = true; out_f32 = false; }
        else if (q.batch != 1 || !allow_table_split) return FACT_ERR_UNSUPPORTED;
    }

    // Up to 56 MB of A and C together, C stays in the memory-side cache (see kStoreThrough); beyond, a program that walks a few such sets of buffers overflows it,
    // and the launches that would have found their operands there lose more (us, streamed / kept, three sets in turn: feed-forward 768 x 3072 of 7288 tokens, 11 + 45 MB,
    // 84.7 / 78.5, 7800 tokens, 12 + 48 MB, 88.3 / 89.5, 8192 tokens, 13 + 50 MB, 81.6 / 88.6; 1024 x 4096 of 5000 tokens, 10 + 41 MB, 98.4 / 98.7, 5600, 11 + 46 MB,
    // 114.7 / 110.7, 6400 118.0 / 119.5; 48 and 64 x 512^3, 25 + 25 and 34 + 34 MB, 18.0 / 17.8 and 20.9 / 26.0, 256 x 256^3, 34 + 34 MB, 19.1 / 22.6).  The other way round where
    // one set serves every layer: a block of 16 x 1024 tokens of 768, 25 + 100 MB, 311 / 302.  Of the whole call: the parts of a column split store alike (25 calls of two
    // parts above the line, each part by its own line or both by the call's: level, 0.99-1.01).
    const int store_stream = q.store_stream >= 0 ? q.store_stream : (double)q.batch * q.M * (nout + q.K) * 2.0 > 56.0 * (1 << 20);

    // (a registry file's choice, and persistent launches where they are asked for, are taken as they stand)
    if (cfg_id < 0 && pl.cfg >= 0 && !pl.loaded && (split == 0 || split == 1) && group_m <= 0 && pl.split == 1 && tail_g <= 1 && q.batch == 1 &&
        q.M > 64 && !g_persistent.load(std::memory_order_relaxed)) {
        const ColumnSplit sp = column_split(pl, q.M, nout, q.K, q.trans_b, gated);
        if (sp.n1 > 0) {
            const int64_t n2 = nout - sp.n1;
            const uint16_t *B = (const uint16_t *)q.B, *up = gated ? (q.B_up ? (const uint16_t *)q.B_up : B + nout * q.ldb) : nullptr;
            const int64_t skip = q.trans_b ? sp.n1 * q.ldb : sp.n1;
            Problem first = q, rest = q;
            first.store_stream = rest.store_stream = store_stream;
            first.N = gated ? 2 * sp.n1 : sp.n1;
            first.B_up = up;
            rest.N = gated ? 2 * n2 : n2;
            rest.B = B + skip;
            rest.B_up = up ? up + skip : nullptr;
            rest.C = (char *)q.C + sp.n1 * (q.ep.out_f32 ? 4 : 2);
            if (q.ep.bias) rest.ep.bias = (const uint16_t *)q.ep.bias + sp.n1;
            if (q.ep.residual) rest.ep.residual = (const uint16_t *)q.ep.residual + sp.n1;
            rc = run(first, pl.cfg, 1, pl.group_m, allow_table_split, ws, ws_bytes, stream, route);
            return rc != FACT_OK ? rc : run(rest, sp.cfg, 1, 0, allow_table_split, ws, ws_bytes, stream, route);
        }
    }

    GemmArgs a;
    std::memset(&a, 0, sizeof a);
    a.A = (const __bf16 *)q.A;
    a.B = (const __bf16 *)q.B;
    a.B_up = gated ? (q.B_up ? (const __bf16 *)q.B_up : (const __bf16 *)q.B + nout * q.ldb) : nullptr;
    a.C = (__bf16 *)q.C;
    a.bias = (const __bf16 *)q.ep.bias;
    a.res = (const __bf16 *)q.ep.residual;
    a.lda = q.lda; a.ldb = q.ldb; a.ldc = q.ldc; a.ldr = q.ep.ldr;
    a.stride_a = q.stride_a; a.stride_b = q.stride_b; a.stride_c = q.stride_c; a.stride_r = q.ep.stride_r;
    a.M = (int)q.M; a.N = (int)q.N; a.K = (int)q.K;
    a.act = q.ep.act;
    a.splits = 1;
    a.group_m = pl.group_m;
    // 16-byte vector access to C / residual / bias in the epilogue
    a.out_f32 = out_f32 ? 1 : 0;
    a.c_f32 = c_f32 ? 1 : 0;
    a.f16 = q.ep.f16;
    // (an fp32 row of 8 columns is two 16-byte pieces: ldc and the batch stride in multiples of 4)
    a.vec_store = (nout % 8 == 0) && q.ldc % (c_f32 ? 4 : 8) == 0 && aligned16(q.C) && q.stride_c % (c_f32 ? 4 : 8) == 0 &&
                  (!q.ep.bias || aligned16(q.ep.bias)) &&
                  (!q.ep.residual || (aligned16(q.ep.residual) && q.ep.ldr % 8 == 0 && q.ep.stride_r % 8 == 0)) &&
                  q.ldc < ((int64_t)1 << 21) && q.ep.ldr < ((int64_t)1 << 21);     // a tile's rows within 2^31 bytes: 32-bit row offsets in the epilogue

    const int unit = gated ? 64 : 32;                 // elements of C between the addresses that rows may begin at (see kStoreThrough)
    a.store_through = ((uintptr_t)q.C & (uintptr_t)(2 * unit - 1)) == 0 && q.ldc % unit == 0 && (q.batch == 1 || q.stride_c % unit == 0);

    a.store_stream = store_stream;

    hipError_t e;
    if (pl.cfg < 0) {
        if (cfg_id != FACT_CONFIG_GUARDED && ragged_serves(a, q.trans_b != 0, q.batch)) {
            const int form = ragged_form(a, q.trans_b != 0, q.batch);
            if (route) return route->add(FACT_ROUTE_RAGGED, form, q.N);
            e = launch_ragged_gemm(a, q.trans_b != 0, form, (int)q.batch, stream);
            return e == hipSuccess ? FACT_OK : hip_fail(e, "ragged gemm launch");
        }
        if (route) return route->add(FACT_ROUTE_GUARDED, -1, q.N);
        e = launch_fallback_gemm(a, q.trans_b != 0, (int)q.batch, stream);
        return e == hipSuccess ? FACT_OK : hip_fail(e, "fallback gemm launch");
    }

    const ConfigDesc &c = g_configs[pl.cfg];
    const int bn_out = gated ? c.bn / 2 : c.bn;
    const int64_t tiles_m = (q.M + c.bm - 1) / c.bm, tiles_n = (nout + bn_out - 1) / bn_out;
    if (tiles_m * tiles_n > INT32_MAX / 2) return FACT_ERR_DIM;
    a.tiles_m = (int)tiles_m; a.tiles_n = (int)tiles_n;

    a.pf_dist = 1;
    a.tail_first = (int)(tiles_m * tiles_n);
    if (tail_g > 1 && pl.split <= 1) {
        const TailPlan t = tail_plan(c, tiles_m * tiles_n, q.K, tail_g);
        if (t.g > 1 && ws && aligned16(ws) && ws_bytes >= t.bytes()) {
            // flags carry a launch-unique 64-bit value, so the workspace needs no clearing
            a.tail_first = (int)t.first;
            a.tail_g = t.g;
            a.tail_ws = (float *)((char *)ws + t.partials_offset());
            a.tail_flags = (unsigned long long *)((char *)ws + t.flags_offset());
            a.tail_status = (unsigned long long *)ws;
            a.tail_epoch = ++g_tail_epoch;
            a.tail_budget = g_tail_budget.load(std::memory_order_relaxed);
        } else if (split < 0) {
            return t.g > 1 ? FACT_ERR_WORKSPACE : FACT_ERR_UNSUPPORTED;
        }
    }
    if (pl.split > 1) {
        // K ranges are multiples of the 64-element staging step
        int64_t kps = (q.K + pl.split - 1) / pl.split;
        kps = (kps + 63) / 64 * 64;
        const int splits = (int)((q.K + kps - 1) / kps);
        if (splits <= 1) {
            pl.split = 1;
        } else {
            const size_t need = splitk_ws_bytes(q.M, q.N, pl.split);
            if (!ws) return FACT_ERR_WORKSPACE;
            if (!aligned16(ws)) return FACT_ERR_ALIGN;
            if (ws_bytes < need) return FACT_ERR_WORKSPACE;
            a.splits = splits;
            a.k_per_split = (int)kps;
            a.P = (float *)ws;
        }
    }
    // Few rows against [N][K] weights or a small output, nothing about the launch asked for by the caller or the registry: the
    // skinny kernel where it is the faster one.  It needs no workspace; what the plan would have needed has been
    // checked above all the same.  (Persistent launches where they are asked for, and a registry file's choice, are taken as
    // they stand; a row of the compiled-in table names the best tile configuration: 512^3 5.5 us there, 4.0 here.)
    if (!(a.splits <= 1 && !a.f16 && persistent_grid(c, tiles_m * tiles_n * q.batch) > 0) && cfg_id < 0 && (split == 0 || split == 1) && group_m <= 0 && !pl.loaded && tail_g <= 1)
        if (const int tile = skinny_choice(a, q.trans_b != 0, q.batch, before_cfg < 0 ? c : g_configs[before_cfg], before_cfg < 0 ? a.splits : before_split, near_us); tile != kNoSkinny) {
        if (out_f32) {
            if (a.splits <= 1) {
                const size_t need = (size_t)q.M * (size_t)q.N * sizeof(float);
                if (!ws) return FACT_ERR_WORKSPACE;
                if (!aligned16(ws)) return FACT_ERR_ALIGN;
                if (ws_bytes < need) return FACT_ERR_WORKSPACE;
            }
            a.out_f32 = 0; a.c_f32 = 1;
        }
        a.splits = 1; a.P = nullptr;
        const int form = skinny_form(a, q.trans_b != 0, q.batch, tile);
        if (route) return route->add(FACT_ROUTE_SKINNY, form, q.N);
        e = launch_skinny_gemm(a, q.trans_b != 0, form, (int)q.batch, stream);
        return e == hipSuccess ? FACT_OK : hip_fail(e, "skinny gemm launch");
    }
    // L2 prefetch (see the kernel).  Many work-groups: the ones resident on an XCD (32 CUs) form a
    // block of gsz tile rows x (resident / gsz) tile columns that share panels; each touches its
    // share one step ahead.  (With few work-groups, e.g. long split-K ranges streamed from HBM,
    // unshared prefetching several steps ahead was measured to be slower than none.)
    {
        const int64_t grid = tiles_m * tiles_n * (a.splits > 1 ? a.splits : q.batch);
        const bool soff_ok = q.trans_b || (q.K * q.ldb * 2 < ((int64_t)1 << 31));
        auto pow2_floor = [](int v) { int r = 1; while (r * 2 <= v) r *= 2; return r; };
        // Also with about one work-group per compute unit when K is long and not split: the panels then
        // come from HBM at least once per launch, and inside a transformer block (weights of several
        // layers between two uses) every time.  Measured with operands rotated out of the memory-side
        // cache: Llama QKV 1052 -> 1260 TFLOP/s, down projection 1130 -> 1235, 4096^3 1243 -> 1330;
        // no gain or a small loss for K = 768, for half-empty grids and for split-K ranges.
        const int64_t wgs = a.tail_g > 1 ? a.tail_first + (tiles_m * tiles_n - a.tail_first) * a.tail_g : grid;
        const bool one_round_long_k = pl.split <= 1 && wgs >= 3 * kNumCU / 4 && q.K >= 2048;
        if (soff_ok && c.has_prefetch()) {
            // (a round and a half of whole-K tiles counts as many: 8192 x 2304 x 768 on 384 tiles of 256 x 192,
            // operands from HBM, 48.0 -> 42.9 us with the prefetch, 37.4 -> 36.9 us from the memory-side cache)
            if (grid >= 2 * kNumCU || (a.splits <= 1 && grid >= 3 * kNumCU / 2) || one_round_long_k) {
                const int gsz = (int)(pl.group_m < tiles_m ? pl.group_m : tiles_m);
                const int resident = 32 * wgs_per_cu(c);
                int sb = pow2_floor(gsz), sa = pow2_floor(resident / gsz > 0 ? resident / gsz : 1);
                if (sa > tiles_n) sa = pow2_floor((int)tiles_n);
                a.pf_sa = sa > 32 ? 32 : sa; a.pf_sb = sb > 32 ? 32 : sb; a.pf_dist = 1;
            }
        }
    }
    if (out_f32 && a.splits <= 1) {                   // one fp32 plane
        const size_t need = (size_t)q.M * (size_t)q.N * sizeof(float);
        if (!ws) return FACT_ERR_WORKSPACE;
        if (!aligned16(ws)) return FACT_ERR_ALIGN;
        if (ws_bytes < need) return FACT_ERR_WORKSPACE;
        a.P = (float *)ws;
    }
    // Persistent launch: more work items than resident work-groups, K whole, no tail split.
    a.persist_items = 0; a.persist_z = 1; a.persist_grid = 0;
    if (a.tail_g <= 1 && a.splits <= 1 && !a.f16) {       // (the persistent form is instantiated for bf16 only)
        const int grid = persistent_grid(c, tiles_m * tiles_n * q.batch);
        if (grid > 0) { a.persist_items = (int)(tiles_m * tiles_n * q.batch); a.persist_z = (int)q.batch; a.persist_grid = grid; }
    }
    if (!grid_fits(c, a.tail_g > 1 ? a.tail_first + (tiles_m * tiles_n - a.tail_first) * a.tail_g : tiles_m * tiles_n)) return FACT_ERR_DIM;
    // (the kernel numbers (K range or batch entry, tile) pairs with 32-bit integers)
    if (tiles_m * tiles_n * (a.splits > 1 ? (int64_t)a.splits : q.batch) > INT32_MAX / 2) return FACT_ERR_DIM;
    if (route) {
        route->add(a.tail_g > 1 ? FACT_ROUTE_TAIL : a.persist_items > 0 ? FACT_ROUTE_PERSISTENT : FACT_ROUTE_TILES, pl.cfg, q.N, a.store_stream);
        return a.splits > 1 || out_f32 ? route->add(FACT_ROUTE_REDUCE, -1, q.N) : FACT_OK;
    }
    e = c.launch(a, q.trans_b != 0, a.splits > 1 ? a.splits : (int)q.batch, stream);
    if (e != hipSuccess) return hip_fail(e, "gemm launch");
    if (a.splits > 1 || out_f32) {
        e = launch_splitk_reduce(a, stream);
        if (e != hipSuccess) return hip_fail(e, "split-K reduce launch");
    }
    return FACT_OK;
}

static fact_epilogue ep_or_none(const fact_epilogue *ep)
{
    fact_epilogue e;
    std::memset(&e, 0, sizeof e);
    if (ep) e = *ep;
    return e;
}

}  // namespace fact

using namespace fact;

extern "C" {

int fact_gemm(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
              int trans_b, void *C, int64_t ldc, const fact_epilogue *ep, void *stream)
{
    Problem q{1, M, N, K, A, lda, 0, B, ldb, 0, trans_b, nullptr, C, ldc, 0, ep_or_none(ep)};
    return run(q, -1, 1, 0, false, nullptr, 0, (hipStream_t)stream);
}

int fact_gemm_batched(int64_t batch, int64_t M, int64_t N, int64_t K,
                      const void *A, int64_t lda, int64_t stride_a,
                      const void *B, int64_t ldb, int64_t stride_b, int trans_b,
                      void *C, int64_t ldc, int64_t stride_c,
                      const fact_epilogue *ep, void *stream)
{
    Problem q{batch, M, N, K, A, lda, stride_a, B, ldb, stride_b, trans_b, nullptr, C, ldc, stride_c, ep_or_none(ep)};
    return run(q, -1, 1, 0, false, nullptr, 0, (hipStream_t)stream);
}

int fact_gemm_splitk(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                     int trans_b, void *C, int64_t ldc, const fact_epilogue *ep,
                     int split_k, void *ws, size_t ws_bytes, void *stream)
{
    if (split_k < 0) return FACT_ERR_UNSUPPORTED;
    Problem q{1, M, N, K, A, lda, 0, B, ldb, 0, trans_b, nullptr, C, ldc, 0, ep_or_none(ep)};
    return run(q, -1, split_k, 0, true, ws, ws_bytes, (hipStream_t)stream);
}

// workspace a plan needs: split-K partial planes, or the partial tiles and flags of a tail split
static size_t plan_ws_bytes(const Plan &pl, int64_t M, int64_t N, int64_t K, bool gated)
{
    if (pl.cfg < 0) return 0;
    if (pl.split > 1) return splitk_ws_bytes(M, N, pl.split);
    if (pl.split < -1) {
        const ConfigDesc &c = g_configs[pl.cfg];
        const int64_t nout = gated ? N / 2 : N, bn_out = gated ? c.bn / 2 : c.bn;
        const int64_t tiles = ((M + c.bm - 1) / c.bm) * ((nout + bn_out - 1) / bn_out);
        return tail_plan(c, tiles, K, -pl.split).bytes();
    }
    return 0;
}

}  // extern "C"

namespace fact {

Workspace splitk_workspace(int64_t M, int64_t N, int64_t K)
{
    size_t least = 0, full = 0;
    // the table's choice may depend on layout and epilogue (gated or not); report the largest over them
    for (int tb = 0; tb < 2; ++tb)
        for (int gated = 0; gated < 2; ++gated) {
            if (gated && (!tb || N % 2)) continue;
            const Plan pl = make_plan(1, M, N, K, tb, gated ? FACT_ACT_SILU_GATE : FACT_ACT_NONE, true);
            const size_t b = plan_ws_bytes(pl, M, N, K, gated != 0), near = splitk_ws_bytes(M, N, pl.near_split);
            if (b > least) least = b;
            if (near > full) full = near;
        }
    return {least, full > least ? full : least};
}

// The two GEMMs of the feed-forward block as planned for any workspace, and what they need.
struct MlpPlans { Plan up, down; Workspace need; };
static MlpPlans mlp_plans(int64_t T, int64_t d_model, int64_t d_ff, int act)
{
    const bool gated = act == FACT_ACT_SILU_GATE;
    MlpPlans p{make_plan(1, T, gated ? 2 * d_ff : d_ff, d_model, 1, act, true), down_plan(T, d_model, d_ff), {}};
    const size_t up = p.up.split < -1 ? plan_ws_bytes(p.up, T, gated ? 2 * d_ff : d_ff, d_model, gated) : 0;   // GEMM 1 never splits K
    const size_t down = plan_ws_bytes(p.down, T, d_model, d_ff, false), near = splitk_ws_bytes(T, d_model, p.down.near_split);
    p.need.least = up > down ? up : down;
    p.need.full = near > p.need.least ? near : p.need.least;
    return p;
}

Workspace mlp_workspace(int64_t T, int64_t d_model, int64_t d_ff, int act) { return mlp_plans(T, d_model, d_ff, act).need; }

}  // namespace fact

extern "C" {

size_t fact_gemm_splitk_workspace_bytes(int64_t M, int64_t N, int64_t K, int split_k)
{
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    if (split_k == 0) return splitk_workspace(M, N, K).full;
    if (split_k > 0) return splitk_ws_bytes(M, N, split_k);
    // forced tail split (fact_gemm_ex): the largest need over the tile configurations
    size_t need = 0;
    for (int i = 0; i < kNumConfigs; ++i)
        for (int gated = 0; gated < 2; ++gated) {
            Plan pl; pl.cfg = i; pl.split = split_k;
            const size_t b = plan_ws_bytes(pl, M, N, K, gated != 0);
            if (b > need) need = b;
        }
    return need;
}

size_t fact_gemm_f32out_workspace_bytes(int64_t M, int64_t N, int64_t K, int split_k)
{
    if (M <= 0 || N <= 0 || K <= 0) return 0;
    int s = split_k < 0 ? 0 : split_k;
    if (s == 0)                                       // the table's split-K factor, over both layouts (tail splits do not apply)
        for (int tb = 0; tb < 2; ++tb) {
            const Plan pl = make_plan(1, M, N, K, tb, FACT_ACT_NONE, true);
            if (pl.cfg >= 0 && pl.most_ranges() > s) s = pl.most_ranges();
        }
    return splitk_ws_bytes(M, N, s);                  // nothing when K stays whole: the main kernel writes the fp32 result
}

int fact_gemm_ex(int64_t batch, int64_t M, int64_t N, int64_t K,
                 const void *A, int64_t lda, int64_t stride_a,
                 const void *B, int64_t ldb, int64_t stride_b, int trans_b,
                 void *C, int64_t ldc, int64_t stride_c,
                 const fact_epilogue *ep, int config_id, int split_k, int group_m,
                 void *ws, size_t ws_bytes, void *stream)
{
    Problem q{batch, M, N, K, A, lda, stride_a, B, ldb, stride_b, trans_b, nullptr, C, ldc, stride_c, ep_or_none(ep)};
    return run(q, config_id, split_k, group_m, true, ws, ws_bytes, (hipStream_t)stream);
}

int fact_test_route(int64_t batch, int64_t M, int64_t N, int64_t K,
                    const void *A, int64_t lda, int64_t stride_a,
                    const void *B, int64_t ldb, int64_t stride_b, int trans_b,
                    void *C, int64_t ldc, int64_t stride_c,
                    const fact_epilogue *ep, int config_id, int split_k, int group_m,
                    void *ws, size_t ws_bytes, int max_launches, int *kinds, int *configs, int64_t *columns)
{
    Problem q{batch, M, N, K, A, lda, stride_a, B, ldb, stride_b, trans_b, nullptr, C, ldc, stride_c, ep_or_none(ep)};
    Route route;
    const int rc = run(q, config_id, split_k, group_m, ws != nullptr, ws, ws_bytes, nullptr, &route);
    if (rc != FACT_OK) return rc;
    g_last_route = route;
    for (int i = 0; i < route.launches && i < max_launches && i < Route::kMax; ++i) {
        if (kinds) kinds[i] = route.kind[i];
        if (configs) configs[i] = route.cfg[i];
        if (columns) columns[i] = route.columns[i];
    }
    return route.launches;
}

int fact_test_route_streams(int max_launches, int *streams)
{
    const Route &route = g_last_route;
    for (int i = 0; i < route.launches && i < max_launches && i < Route::kMax; ++i)
        if (streams) streams[i] = route.streams[i];
    return route.launches;
}

size_t fact_block_mlp_workspace_bytes(int64_t T, int64_t d_model, int64_t d_ff, int act)
{
    if (T <= 0 || d_model <= 0 || d_ff <= 0) return 0;
    if (act < 0 || act > 2) return 0;
    return mlp_workspace(T, d_model, d_ff, act).full;
}

static int block_mlp_impl(int f16, int64_t T, int64_t d_model, int64_t d_ff,
                          const void *X, const void *W1, const void *W1u, const void *b1, int act,
                          const void *W2, const void *b2, const void *R,
                          void *H, void *Y, void *ws, size_t ws_bytes, void *stream)
{
    if (!X || !W1 || !W2 || !H || !Y) return FACT_ERR_NULL;
    if (act != FACT_ACT_NONE && act != FACT_ACT_GELU_TANH && act != FACT_ACT_SILU_GATE) return FACT_ERR_EPILOGUE;
    const bool gated = act == FACT_ACT_SILU_GATE;
    if (gated && !W1u) return FACT_ERR_NULL;
    if (!gated && W1u) return FACT_ERR_EPILOGUE;
    if (gated && b1) return FACT_ERR_EPILOGUE;
    if (T <= 0 || d_model <= 0 || d_ff <= 0) return FACT_ERR_DIM;

    // GEMM 1: H = act(X W1^T + b1); gated: contraction over 2*d_ff columns, gate then up
    fact_epilogue e1;
    std::memset(&e1, 0, sizeof e1);
    e1.bias = b1;
    e1.act = act;
    e1.f16 = f16;
    Problem q1{1, T, gated ? 2 * d_ff : d_ff, d_model, X, d_model, 0, W1, d_model, 0, 1,
               gated ? W1u : nullptr, H, d_ff, 0, e1};
    // GEMM 2: Y = H W2^T + b2 + R  (may split K = d_ff when the table says so and ws allows)
    fact_epilogue e2;
    std::memset(&e2, 0, sizeof e2);
    e2.bias = b2;
    e2.residual = R;
    e2.ldr = d_model;
    e2.act = FACT_ACT_NONE;
    e2.f16 = f16;
    Problem q2{1, T, d_model, d_ff, H, d_ff, 0, W2, d_ff, 0, 1, nullptr, Y, d_model, 0, e2};
    // everything either launch could refuse is checked before the first one: on error nothing runs
    int rc = validate(q1);
    if (rc == FACT_OK) rc = validate(q2);
    if (rc != FACT_OK) return rc;
    const MlpPlans plans = mlp_plans(T, d_model, d_ff, act);
    const size_t need = plans.need.least;
    if (need > 0 && (!ws || ws_bytes < need)) return FACT_ERR_WORKSPACE;
    if (need > 0 && !aligned16(ws)) return FACT_ERR_ALIGN;
    // (the first GEMM never splits K into planes, but its last round of tiles may be split)
    const bool tail = plans.up.split < -1;
    rc = run(q1, -1, tail ? 0 : 1, 0, tail, ws, ws_bytes, (hipStream_t)stream);
    if (rc != FACT_OK) return rc;
    if (need == 0 && !ws) return run(q2, -1, 0, 0, false, nullptr, 0, (hipStream_t)stream);
    return run(q2, -1, 0, 0, true, ws, ws_bytes, (hipStream_t)stream, nullptr, &plans.down);
}

int fact_block_mlp(int64_t T, int64_t d_model, int64_t d_ff,
                   const void *X, const void *W1, const void *W1u, const void *b1, int act,
                   const void *W2, const void *b2, const void *R,
                   void *H, void *Y, void *ws, size_t ws_bytes, void *stream)
{
    return block_mlp_impl(0, T, d_model, d_ff, X, W1, W1u, b1, act, W2, b2, R, H, Y, ws, ws_bytes, stream);
}

int fact_block_mlp_f16(int64_t T, int64_t d_model, int64_t d_ff,
                       const void *X, const void *W1, const void *W1u, const void *b1, int act,
                       const void *W2, const void *b2, const void *R,
                       void *H, void *Y, void *ws, size_t ws_bytes, void *stream)
{
    return block_mlp_impl(1, T, d_model, d_ff, X, W1, W1u, b1, act, W2, b2, R, H, Y, ws, ws_bytes, stream);
}

int fact_num_configs(void) { return kNumConfigs; }

int fact_config_info(int id, int *tile_m, int *tile_n, int *waves_m, int *waves_n, int *lds_bytes)
{
    if (id < 0 || id >= kNumConfigs) return FACT_ERR_UNSUPPORTED;
    const ConfigDesc &c = g_configs[id];
    if (tile_m) *tile_m = c.bm;
    if (tile_n) *tile_n = c.bn;
    if (waves_m) *waves_m = c.wm;
    if (waves_n) *waves_n = c.wn;
    if (lds_bytes) *lds_bytes = c.lds_bytes();
    return FACT_OK;
}

int fact_select_config(int64_t batch, int64_t M, int64_t N, int64_t K, int trans_b, int act,
                       int *config_id, int *split_k)
{
    if (batch <= 0 || M <= 0 || N <= 0 || K <= 0) return FACT_ERR_DIM;
    if (trans_b != 0 && trans_b != 1) return FACT_ERR_LAYOUT;
    if (act < 0 || act > 2) return FACT_ERR_EPILOGUE;
    if (act == FACT_ACT_SILU_GATE && (N % 2 || !trans_b)) return FACT_ERR_EPILOGUE;
    const Plan pl = make_plan(batch, M, N, K, trans_b, act, true);
    if (config_id) *config_id = pl.near_cfg >= 0 ? pl.near_cfg : pl.cfg;
    if (split_k) *split_k = pl.near_cfg >= 0 ? pl.near_split : pl.split;
    return FACT_OK;
}

int fact_persistent_grid(int64_t batch, int64_t M, int64_t N, int64_t K, int trans_b, int act, int config_id)
{
    if (batch <= 0 || M <= 0 || N <= 0 || K <= 0) return 0;
    if (config_id < 0) {
        Plan pl = make_plan(batch, M, N, K, trans_b, act, false);
        if (pl.split != 1) return 0;
        config_id = pl.near_cfg >= 0 ? pl.near_cfg : pl.cfg;
    }
    if (config_id < 0 || config_id >= kNumConfigs) return 0;
    const ConfigDesc &c = g_configs[config_id];
    const int64_t nout = act == FACT_ACT_SILU_GATE ? N / 2 : N;
    const int bn_out = act == FACT_ACT_SILU_GATE ? c.bn / 2 : c.bn;
    return persistent_grid(c, ((M + c.bm - 1) / c.bm) * ((nout + bn_out - 1) / bn_out) * batch);
}

const char *fact_status_string(int status)
{
    switch (status) {
    case FACT_OK: return "ok";
    case FACT_ERR_NULL: return "required pointer is NULL";
    case FACT_ERR_DIM: return "bad dimension, leading dimension or stride";
    case FACT_ERR_ALIGN: return "pointer alignment";
    case FACT_ERR_LAYOUT: return "bad layout flag";
    case FACT_ERR_EPILOGUE: return "bad epilogue";
    case FACT_ERR_WORKSPACE: return "workspace missing or too small";
    case FACT_ERR_UNSUPPORTED: return "unsupported configuration";
    case FACT_ERR_HIP: return "HIP error";
    default: return "unknown status";
    }
}

// ---- split-K without a caller's workspace: partials in a library-owned static device array --------
// For callers that cannot allocate (code under graph capture, serving loops, harnesses that forbid
// it).  The array lives in this library's device image: every GPU the library runs on holds its own
// copy, at its own address, until the process ends.  Host code never uses the array's name as an
// address (on the host it is a stand-in for the symbol): the address is asked for once per device,
// with that device current, and kept.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static constexpr int kMaxDevices = 64;
static std::atomic<void *> g_scratch_ptr[kMaxDevices];

static int static_scratch(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "static scratch: hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return FACT_ERR_UNSUPPORTED;
    void *ptr = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!ptr) {
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));       // this device's copy (the current device)
        if (e != hipSuccess || !ptr) return hip_fail(e, "static scratch: hipGetSymbolAddress");
        g_scratch_ptr[dev].store(ptr, std::memory_order_release); // (two threads may both ask: they get the same address)
    }
    *out = ptr;
    return FACT_OK;
}

size_t fact_gemm_splitk_static_capacity(void) { return kStaticScratchBytes; }

int fact_gemm_splitk_static_init(void)
{
    void *ptr = nullptr;
    return static_scratch(&ptr);
}

int fact_gemm_splitk_static(int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
                            int trans_b, void *C, int64_t ldc, const fact_epilogue *ep, int split_k, void *stream)
{
    if (split_k < 0) return FACT_ERR_UNSUPPORTED;
    if (M <= 0 || N <= 0 || K <= 0) return FACT_ERR_DIM;
    // what fact_gemm_splitk would ask the caller for, for this very call (layout and epilogue known here)
    const fact_epilogue e0 = ep_or_none(ep);
    Plan pl = make_plan(1, M, N, K, trans_b, e0.act, true);
    if (split_k > 0) pl.split = split_k;
    const bool gated = e0.act == FACT_ACT_SILU_GATE;
    size_t need = pl.split > 1 && e0.out_f32 ? splitk_ws_bytes(M, N, pl.split) : plan_ws_bytes(pl, M, N, K, gated);
    if (need > kStaticScratchBytes) {
        std::snprintf(g_last_error, sizeof g_last_error,
                      "fact_gemm_splitk_static: this call needs %zu bytes of partial sums, the static array holds %zu "
                      "(use fact_gemm_splitk with a workspace, or a smaller split_k)", need, kStaticScratchBytes);
        return FACT_ERR_WORKSPACE;
    }
    void *ptr = nullptr;
    const int rc = static_scratch(&ptr);
    if (rc != FACT_OK) return rc;
    Problem q{1, M, N, K, A, lda, 0, B, ldb, 0, trans_b, nullptr, C, ldc, 0, e0};
    return run(q, -1, split_k, 0, true, ptr, kStaticScratchBytes, (hipStream_t)stream);
}

int fact_tail_timeouts(const void *ws, void *stream, int *gave_up)
{
    if (!ws || !gave_up) return FACT_ERR_NULL;
    if ((uintptr_t)ws & 15u) return FACT_ERR_ALIGN;
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "fact_tail_timeouts: stream synchronize");
    unsigned long long word = 0;
    e = hipMemcpy(&word, ws, sizeof word, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return hip_fail(e, "fact_tail_timeouts: read of the status word");
    const unsigned long long last = g_tail_epoch.load();
    // epochs handed out by this process: (first, last], compared modulo 2^64
    *gave_up = (word - g_tail_epoch_first - 1) < (last - g_tail_epoch_first) ? 1 : 0;
    return FACT_OK;
}

void fact_test_tail_poll_budget(int polls) { g_tail_budget.store(polls, std::memory_order_relaxed); }
int fact_tune_persistent(int mode) { return fact::g_persistent.exchange(mode != 0 ? 1 : 0, std::memory_order_relaxed); }

// Registry file: text, one entry per line (see include/fact.h).  Entries of another rule, data type
// or architecture are skipped, as are entries naming a configuration this build does not have or
// one that does not serve the entry's layout.
int fact_registry_load(const char *path)
{
    if (!path) return FACT_ERR_NULL;
    std::FILE *f = std::fopen(path, "r");
    if (!f) return FACT_ERR_UNSUPPORTED;
    char line[1024];
    bool header = false;
    std::vector<TableRow> rows;
    while (std::fgets(line, sizeof line, f)) {
        if (line[0] == '#') {
            int ver = 0;
            if (std::sscanf(line, "# fact-registry %d", &ver) == 1) {
                if (ver != 1) { std::fclose(f); return FACT_ERR_UNSUPPORTED; }
                header = true;
            }
            continue;
        }
        if (!header) { std::fclose(f); return FACT_ERR_UNSUPPORTED; }      // entries before the format line
        char rule[32], dtype[32], arch[32], layout[8], epi[16];
        long long batch, M, N, K;
        int cfg, split, group_m;
        if (std::sscanf(line, "%31s %31s %31s %lld %lld %lld %lld %7s %15s %d %d %d", rule, dtype, arch, &batch, &M, &N, &K,
                        layout, epi, &cfg, &split, &group_m) != 12)
            continue;
        if (std::strcmp(rule, "gemm") || std::strcmp(dtype, "bf16") || std::strcmp(arch, "gfx950")) continue;
        const int trans_b = !std::strcmp(layout, "nk") ? 1 : !std::strcmp(layout, "kn") ? 0 : -1;
        const int gated = !std::strcmp(epi, "gated") ? 1 : !std::strcmp(epi, "plain") ? 0 : -1;
        if (trans_b < 0 || gated < 0 || batch < 1 || M < 1 || N < 1 || K < 1) continue;
        if (cfg < 0 || cfg >= kNumConfigs || !g_configs[cfg].serves(trans_b) || (gated && !g_configs[cfg].gate_capable())) continue;
        if (split == 0 || split == -1 || split > kMaxGridZ || group_m < 0) continue;
        rows.push_back(TableRow{batch, M, N, K, trans_b, gated, cfg, split, group_m});
    }
    std::fclose(f);
    if (!header) return FACT_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_registry_mutex);
    g_registry.insert(g_registry.begin(), rows.begin(), rows.end());       // the newest load is consulted first
    return (int)rows.size();
}

void fact_registry_clear(void)
{
    std::lock_guard<std::mutex> lock(g_registry_mutex);
    g_registry.clear();
}

int fact_registry_size(void)
{
    std::lock_guard<std::mutex> lock(g_registry_mutex);
    return (int)g_registry.size();
}

const char *fact_last_error(void) { return g_last_error; }

int fact_version(void) { return 205; }

}  // extern "C"
