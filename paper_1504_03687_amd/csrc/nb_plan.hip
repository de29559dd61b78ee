// Launch plans of the regular-force kernels: which mapping, how many rows
// per lane or per wave, and how many contiguous j-splits.  These rules shape
// every force launch (and so its memory traffic); the rest of the runtime is
// in nb_runtime.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "nbreg.h"
#include "nb_internal.h"
#include "nb_runtime.h"

using nb::Plan;

namespace nbrt {

int64_t bucket_log2(int64_t v)
{
    int64_t b = 0;
    while ((int64_t(1) << (b + 1)) <= v) ++b;
    return b;
}

// Whether a row-per-lane launch (mapping 1, one row per lane) packs the j-set
// and runs the scalar-operand kernel.  The pack costs a launch and a copy of
// the j-set (about 3 us at n = 131072, 25 us at 2^20), and a wave alone on its
// SIMD waits longer for scalar loads than for LDS, so the block has to be
// large enough to repay both: above 2^26 pairs from 1024 rows on, above 2^27
// from 512.  Whole calls, LDS against packed, mixed / FP64: 16384 rows of 131072
// 1959 / 2735 against 1812 / 2487 us, 1024 of 131072 157 / 188 against 153 / 184,
// 2048 of 65536 159 / 193 against 151 / 187, 8000 of 16384 158 / 197 against 152
// / 195, 5000 of 16384 117 / 141 against 112 / 131, 9000 of 9000 117 / 142 against
// 113 / 135, 1100 of 65536 109 / 125 against 109 / 122; with fewer rows 900 of
// 131072 149 / 176 against 151 / 179, 550 of 131072 104 / 116 against 112 / 123;
// 256 of 2^20 260 / 351 against 280 / 365.
bool pack_pays(int mapping, int rows_per_lane, int64_t n, int32_t n_i)
{
    return mapping == 1 && rows_per_lane == 1 && n_i >= 512 &&
           n * (int64_t)n_i > (int64_t(1) << (n_i >= 1024 ? 26 : 27));
}

// Row groups of a launch: waves in mappings 2 and 3, work-groups of four
// waves in mapping 1.
static int64_t row_groups(int32_t n_i, int mapping, int rows)
{
    const int64_t per = mapping == 2 ? rows : mapping == 3 ? nb::kWave : (int64_t)rows * nb::kBlock;
    return std::max<int64_t>(1, (n_i + per - 1) / per);
}

// Bodies of the shortest useful split: 256 in the wave mapping, 512 in the
// packed launches, whose blocks have enough row tiles, and 64 in the
// row-per-lane mappings through LDS: a lane is a serial chain of its split's
// pairs, so small blocks want short splits, at the price of a record per
// split and row in the merge.  32 (the run of the folds) where splits of 64
// come to at most one wave per SIMD: whole calls, splits of 64 against 32,
// FP64 / mixed, 1024 rows of 1024 24.0 / 36.0 against 17.4 / 29.8 us, 256 of
// 4096 22.7 / 32.3 against 18.3 / 28.1, 1024 of 4096 (one wave per SIMD) 26.4
// / 38.6 against 24.7 / 37.6; past that it loses, 4096 of 4096 (four waves)
// 46.6 / 51.2 against 50.3 / 58.3.  128 above kShortSplitBodies bodies, whose
// splits of 64 would be more than 2048 a row: splits of 64 against 128, 41 rows
// of 200000 37.0 / 34.0 against 34.8 / 31.8 us, 41 of 262144 41.7 / 40.0 against
// 37.6 / 36.8, 64 of 262144 44.0 / 41.9 against 39.8 / 40.7, 100 of 262144 62.0 /
// 57.0 against 57.0 / 54.3; 41 of 131072 26.8 / 33.8 against 27.2 / 34.4, 64 of
// 131072 28.0 / 27.0 against 28.8 / 28.0.
constexpr int64_t kShortSplitBodies = 131072;

static int64_t min_split(const nb_ctx *ctx, int64_t n, int32_t n_i, int mapping, int rows)
{
    if (mapping == 2) return 4 * nb::kWave;
    if (pack_pays(mapping, rows, n, n_i)) return 2 * nb::kTile;
    if (n > kShortSplitBodies) return 2 * nb::kWave;
    const int64_t simds = 4 * (int64_t)(ctx->cu_count > 0 ? ctx->cu_count : 256);
    const int64_t waves = row_groups(n_i, mapping, rows) * (mapping == 1 ? nb::kBlock / nb::kWave : 1) *
                          ((n + nb::kWave - 1) / nb::kWave);
    return waves <= simds ? nb::kFold : nb::kWave;
}

// Largest useful split count.
int64_t max_splits(const nb_ctx *ctx, int64_t n, int32_t n_i, int mapping, int rows)
{
    const int64_t unit = min_split(ctx, n, n_i, mapping, rows);
    return std::max<int64_t>(1, (n + unit - 1) / unit);
}

// Split count of the automatic plan for a given mapping and rows per lane
// (or per wave).
//  * mapping 2 (small blocks stream the j-set): about 2 waves per SIMD in
//    total, and at most kWaveMaxSplits splits per row; more splits only add
//    merge work (measured at N = 2^20, n_i = 1 .. 255).
//  * row per lane through LDS (mapping 3 with 64 rows a work-group, mapping 1
//    with 256): about 8 waves per SIMD in total, down to min_split bodies per split,
//    at most kRowWaveMaxSplits splits.
//    A lane that is alone on its SIMD takes 150 to 200 ns per pair, so long
//    splits leave the chip waiting for few waves.  Whole calls, FP64, with
//    splits of 512 bodies against 64: 1024 rows of 1024 175 against 23 us, 256
//    of 4096 136 against 23, 1024 of 16384 107 against 47 (128 splits 44), 4096
//    of 16384 131 against 112, 256 of 131072 118 against 62 (1024 splits 59).
//  * packed launches: many short waves even out their run-time differences, but
//    every split adds a record per row to the merge: about 32 waves per SIMD,
//    64 above 2^32 pairs.  FP64, per 32768 / 65536 waves: 16001 rows of 100003
//    1826 / 1874 us, 16384 of 131072 2400 / 2508, 4096 of 2^20 4771 / 4782,
//    16384 of 2^20 18946 / 18683, 65536 of 2^20 74216 / 73426.
constexpr int64_t kWaveMaxSplits = 1024;
constexpr int64_t kRowWaveMaxSplits = 4096;

// Split length of a packed launch that its least length of 512 bounds, from 256
// to 1024 in steps of 64 bodies: the one whose work-groups fill the CUs best.
// Cost in pairs of the whole chip: the work-groups of the fullest CU and one more
// for the end of the launch, where few waves are left on each SIMD, each of
// kBlock rows by the split's bodies; and 40 a record for the merge.  It orders
// whole calls as they were measured: 4099 rows of 131072, splits of 512 (16.25
// work-groups per CU) 501 us mixed and 655 FP64, 768 (10.9) 491 and 633, 1024
// (8.1) 535 and 685, 1280 538 and 678, 2048 (4.06) 632 and 785.  (100 a record:
// 1500 of 131072 211 and 269, with 40 203 and 261.)  Not to less than kMinPerCu
// work-groups per CU: at little more than fit at once (10000 of 30000, 6.6 per
// CU instead of 9.1) the last ones run alone, 312 us against 290.  Nor past
// kWave splits where 512 gives no more, which a row's wave merges in one turn
// (10000 of 30000 291 and 402 us with 59, 300 and 410 with 94); but blocks that
// come to fewer than kMinPerCu at the shortest length of those take 256 however
// many splits that is: 2500 of 30000 109 and 124 us with 118, 131 and 151 with
// 59, 4099 of 24576 136 and 163 with 96, 146 and 173 with 64 of 384, 4099 of
// 32768 163 and 200 with 128, 185 and 222 with 64; 6000 of 17000 136 and 165
// with 67, 131 and 156 with 54 is the largest loss.  Whole calls with 512 and with this rule, mixed / FP64: 9000 of
// 16384 188 / 237 and 167 / 217 us, 3000 of 50000 185 / 228 and 164 / 210, 2049
// of 65544 185 / 220 and 163 / 200, 1500 of 200000 321 / 412 and 302 / 393, 4099
// of 131072 501 / 646 and 487 / 627, 7000 794 / 1065 and 771 / 1030; 4000 of
// 65536 261 / 340 and 258 / 343.
// Longer splits, whose number is the target's, gain nothing reliable by it (2222
// of 2^20 1858 and 1896, 3333 2820 and 2775 us).
static int64_t even_split_len(int64_t cus, int64_t n, int32_t n_i)
{
    constexpr int64_t kWaves = nb::kBlock / nb::kWave, kMinPerCu = 10, kLeast = nb::kTile;
    const int64_t tiles = ((int64_t)n_i + nb::kWave - 1) / nb::kWave;
    int64_t best = kLeast, least = INT64_MAX;
    for (int64_t l = kLeast; l <= 4 * kLeast; l += nb::kWave) {
        const int64_t s = (n + l - 1) / l;
        if (s > nb::kWave && n <= 2 * nb::kTile * (int64_t)nb::kWave) continue;
        const int64_t per_cu = ((tiles * s + kWaves - 1) / kWaves + cus - 1) / cus;
        if (per_cu < kMinPerCu) break;
        const int64_t cost = (per_cu + 1) * cus * nb::kBlock * l + n_i * s * 40;
        if (cost < least) {
            least = cost;
            best = l;
        }
    }
    return best;
}

int64_t default_splits(const nb_ctx *ctx, int64_t n, int32_t n_i, int mapping, int rows)
{
    const int64_t cus = ctx->cu_count > 0 ? ctx->cu_count : 256;
    const bool packed = pack_pays(mapping, rows, n, n_i);
    const int64_t u = row_groups(n_i, mapping, rows);
    // in row groups
    const int64_t target = cus * (mapping == 2   ? 8
                                  : mapping == 3 ? 32
                                  : !packed      ? 8
                                  : n * (int64_t)n_i > (int64_t(1) << 32) ? 64 : 32);
    // mapping 2 rounds down: with only ~2 work-groups per CU, one wave group
    // past the target puts a third work-group on some CU and stretches the
    // whole launch by half (72 rows at N = 2^20: 2052 waves took 257 us,
    // against 152 us for 64 rows in 2048 waves).  finish_plan can only lower
    // the count further.  The others round up: at many waves per CU one extra
    // costs little.
    int64_t s = mapping == 2 ? std::max<int64_t>(1, target / u) : (target + u - 1) / u;
    // mapping 2 with few row groups: at most kWaveMaxSplits splits.  Each
    // split adds a partial to every row's merge, which one work-group reads;
    // with bodies loaded four iterations ahead, one wave per SIMD streams the
    // j-set as fast as two.  FP64, N = 2^20, forced plans: 1 row 20.6 us at
    // 2048 splits, 19.7 at 1024, 21.1 at 512; 4 rows 29.1 / 25.6 / 31.9 us.
    // mapping 3, 64 rows of 2^20: 107 us at 4096 splits, 114 at 8192.
    if (mapping == 2) s = std::min(s, kWaveMaxSplits);
    if (mapping != 2) s = std::min(s, kRowWaveMaxSplits);
    s = std::max<int64_t>(1, std::min(s, max_splits(ctx, n, n_i, mapping, rows)));
    return s;
}

// Plan::step of a split count chosen for a launch: the coarsest that can give
// that many splits.
int split_step(int mapping, int64_t splits, int64_t n)
{
    if (mapping == 2) return 0;
    if (splits > (n + nb::kWave - 1) / nb::kWave) return nb::kFold;
    return mapping == 1 && splits * nb::kTile > n ? nb::kWave : 0;
}

// Mappings of the automatic plan by block size, from steady-state whole calls:
//  * wave mapping (rows in scalar registers, lanes over j) up to
//    kWaveMaxRows: 32 rows of 2^20 67.6 us FP64, against 104.7 us with
//    one-wave row-per-lane work-groups (half their lanes idle);
//  * mapping 1 with its scalar-operand kernel where that pays (pack_pays);
//  * between, through LDS: work-groups of 256 rows (mapping 1), or of one wave
//    and 64 rows (mapping 3) where 256-row tiles would hold more than 1.2
//    times the rows of 64-row ones.  Per filled lane the two are alike, the
//    larger work-groups load each body once for four waves: 256 rows of 2^20
//    260 / 351 us mixed / FP64 in mapping 1, 265 / 345 in mapping 3.
constexpr int32_t kWaveMaxRows = 40;

// Largest block whose mixed-precision request runs the FP64 kernels in the
// automatic plan: the wave mapping, which is bound by memory latency, so its
// FP64 kernel is no slower than the mixed one, and it needs no refinement
// launch (nor, for a flagged row, the refinement itself).  N = 2^20, mixed vs
// FP64 wave kernels: 1 row 22.7 vs 20.4 us, 8 rows 36.7 vs 31.4, 32 rows
// 124.7 (one row refined) vs 67.3.  From 64 rows up the mixed one-wave
// row-per-lane kernel is ahead (87 against the FP64 wave kernel's 137 us).
// The results of such a call meet the FP64 bar.
constexpr int32_t kMixedAsF64MaxRows = kWaveMaxRows;

// Automatic plan for a block of n_i rows against n bodies: the autotuned
// entry for the size buckets if there is one (mapping 0: the tuner found none
// faster), else the mapping for its size (above).
Plan auto_plan(const nb_ctx *ctx, int64_t n, int32_t n_i, bool mixed)
{
    auto it = ctx->tuned.find(std::make_tuple((int)mixed, bucket_log2(n), bucket_log2(n_i)));
    if (it != ctx->tuned.end() && it->second.mapping != 0) {
        Plan p = it->second;
        p.step = split_step(p.mapping, p.splits, n);
        return p;
    }
    if (mixed && n_i <= kMixedAsF64MaxRows) {
        Plan p = auto_plan(ctx, n, n_i, false);
        p.f64 = 1;
        return p;
    }
    Plan p{};
    p.rows_per_lane = 1;
    if (n_i <= kWaveMaxRows) {
        p.mapping = 2;
        p.rows_per_lane = n_i >= 4 ? 4 : (n_i >= 2 ? 2 : 1);
    } else {
        const int64_t pad1 = ((int64_t)n_i + nb::kBlock - 1) / nb::kBlock * nb::kBlock;
        const int64_t pad3 = ((int64_t)n_i + nb::kWave - 1) / nb::kWave * nb::kWave;
        const bool packed = pack_pays(1, 1, n, n_i);
        p.mapping = !packed && pad1 * 5 > pad3 * 6 ? 3 : 1;
        // the least split, but no coarser than a wave: 300 rows of 262144 take 1366
        // splits of 192 bodies (117 us mixed), not 1024 of 256 (124)
        if (!packed)
            p.step = (int)std::min<int64_t>(min_split(ctx, n, n_i, p.mapping, p.rows_per_lane),
                                            nb::kWave);
    }
    p.splits = (int)default_splits(ctx, n, n_i, p.mapping, p.rows_per_lane);
    // packed launches with splits of the least length: their number only falls
    // out of it
    if (pack_pays(p.mapping, p.rows_per_lane, n, n_i) &&
        p.splits == max_splits(ctx, n, n_i, p.mapping, p.rows_per_lane)) {
        const int64_t len = even_split_len(ctx->cu_count > 0 ? ctx->cu_count : 256, n, n_i);
        p.splits = (int)((n + len - 1) / len);
        p.step = nb::kWave;
    }
    return p;
}

// Normalises a plan for (n, n_i): fills zero fields, rounds split lengths.
void finish_plan(Plan &p, int64_t n, int32_t n_i, int64_t *split_len)
{
    if (p.splits < 1) p.splits = 1;
    const int64_t unit = p.step ? p.step : p.mapping == 1 ? nb::kTile : nb::kWave;
    const int64_t units = (n + unit - 1) / unit;
    int64_t per = (units + p.splits - 1) / p.splits;
    if (per < 1) per = 1;
    *split_len = per * unit;
    p.splits = (int)((n + *split_len - 1) / *split_len);
    if (p.splits < 1) p.splits = 1;
    if (p.mapping == 1 && p.splits > 65535) {   // grid.y limit
        *split_len = ((n + 65534) / 65535 + unit - 1) / unit * unit;
        p.splits = (int)((n + *split_len - 1) / *split_len);
    }
    (void)n_i;
}

// Fewest splits that a call without room for its plan's is lowered to: splits of
// 512 bodies, or of 128 in one-wave work-groups, as many as still put 16 waves
// on each SIMD (4 of the one-wave work-groups).  With fewer most of the chip
// would idle, so the call is refused instead.
int least_splits(const nb_ctx *ctx, int64_t n, int32_t n_i, const Plan &p)
{
    if (p.mapping == 2) return p.splits;
    const int64_t cus = ctx->cu_count > 0 ? ctx->cu_count : 256;
    const int64_t u1 = row_groups(n_i, 1, 1), u3 = row_groups(n_i, 3, 1);
    const bool narrow = u1 * nb::kBlock * 5 > u3 * nb::kWave * 6;
    const int64_t unit = narrow ? nb::kWave : nb::kTile;
    const int64_t s = std::min(narrow ? (16 * cus + u3 - 1) / u3 : (64 * cus + u1 - 1) / u1,
                               (n + 2 * unit - 1) / (2 * unit));
    const int64_t len = ((n + unit - 1) / unit + s - 1) / s * unit;
    return (int)std::min<int64_t>(p.splits, (n + len - 1) / len);
}

// The plan and its scratch within 'budget' bytes: what does not fit shrinks the
// refinement's chunk partials to an eighth of the budget first (rows past them
// are summed one work-group each, to the same bits; with half of the budget for
// them the splits of 1272 rows of 2^20 fell to 62 in the fixed workspace, 2665
// us mixed against 1558 with 100), then the split count down to 'least', then
// the partials further; the packed j-set takes what is left, if that is enough.
// total() > budget: not even the least fits.
ForceScratch fit_scratch(const nb_ctx *ctx, int64_t n, int32_t n_i, const Plan &wanted,
                         bool refine, int least, size_t budget)
{
    ForceScratch f{};
    f.p = wanted;
    finish_plan(f.p, n, n_i, &f.split_len);
    f.rcap = ctx->redo_rows_limit;
    f.redo = refine ? nb::redo_scratch_bytes(n_i, n, f.rcap) : 0;
    f.slots = nb::force_scratch_bytes(f.p, n_i);
    const size_t pack = pack_pays(f.p.mapping, f.p.rows_per_lane, n, n_i) ? nb::packed_bytes(n) : 0;
    f.pack = pack;
    if (f.total() <= budget) {
        f.least = f.total() == 0;
        return f;
    }
    f.pack = 0;
    auto shrink_redo = [&](size_t most) {
        if (f.redo > most && f.rcap == 0) f.rcap = n_i;
        while (f.redo > most && f.rcap > 0) {
            f.rcap = f.rcap > 1 ? f.rcap / 2 : -1;
            f.redo = nb::redo_scratch_bytes(n_i, n, f.rcap);
        }
    };
    shrink_redo(budget / 8);
    const size_t room = budget > f.redo ? budget - f.redo : 0;
    const size_t per_split = (nb::kSlotComp * sizeof(double) + sizeof(int32_t) +
                              nb::kSegCap * sizeof(int32_t)) * (size_t)std::max(n_i, 1);
    while (f.p.splits > least && f.slots > room) {
        int64_t s = std::max<int64_t>(
            least, std::min<int64_t>((int64_t)(room / per_split), f.p.splits - 1));
        // few waves per SIMD: no more splits than fill the SIMDs evenly.  In the 64
        // MiB of the fixed workspace, FP64, as many as fit / this rule: 1024 rows of
        // 131072 244 us (548 work-groups) / 192 (512, two per CU), 2048 of 65536 251
        // / 200, 4099 of 131072 881 / 775, 16384 of 131072 3647 / 2900, 1272 of 2^20
        // 2217 / 1812; the one loss seen: 10000 of 30000 mixed 395 / 424.
        const int64_t u = row_groups(n_i, f.p.mapping, f.p.rows_per_lane);
        const int64_t at_once = (f.p.mapping == 1 ? 1 : 4) *
                                (int64_t)(ctx->cu_count > 0 ? ctx->cu_count : 256);
        const int64_t k = (u * s + at_once - 1) / at_once, even = (k - 1) * at_once / u;
        if (even >= std::max(1, least) && (k - 1) * ((n + even - 1) / even) < k * ((n + s - 1) / s))
            s = even;
        f.p.splits = (int)std::max<int64_t>(1, s);
        finish_plan(f.p, n, n_i, &f.split_len);
        f.slots = nb::force_scratch_bytes(f.p, n_i);
    }
    if (f.slots + f.redo > budget) shrink_redo(budget > f.slots ? budget - f.slots : 0);
    // few waves per SIMD wait for scalar loads; blocks of many row tiles gain all the
    // same (in the fixed workspace, mixed, LDS / packed: 1500 rows of 100003 205 /
    // 229 us, 2048 of 65536 177 / 191, 10000 of 30000 424 both, 50000 of 50000 3785
    // / 3582; 16384 of 16384 FP64 429 / 416)
    const bool lowered = f.p.splits < wanted.splits;
    if (f.total() + pack <= budget && !(lowered && n_i < 4096)) f.pack = pack;
    f.least = f.p.splits <= least && f.pack == 0 && (f.redo == 0 || f.rcap < 0);
    return f;
}

}  // namespace nbrt
