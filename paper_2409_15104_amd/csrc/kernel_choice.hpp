// Which kernel a call runs on and how its work is cut, as functions of the call's sizes and the number of compute units.
// Plain C++ without HIP, so that a test can ask what a call of given sizes runs on.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace pec {

constexpr int kBM = 256;       // query rows per workgroup of fwd_il_kernel and fwd_simple_kernel
constexpr int kDecWaves = 4;   // KV heads per workgroup of decode_kernel
constexpr int64_t kStaticScratchBytes = 8 << 20;                        // of pec_decode_splitkv_static
constexpr int64_t kStaticPartials = kStaticScratchBytes / (129 * 4);    // (range, query head) pairs that fit: O and LSE in fp32

// The 256 rows of a fwd_il_kernel work item: as many heads of a KV group as divide it, up to 8, and 256 / heads query
// positions of each.  All of them read the same keys, so the choice changes no traffic; fewer positions waste less at
// the causal diagonal (a workgroup walks to the last key of its last row) and in the last, partly filled row tile.  256
// prompts of the benchmark's length mix with 32 q / 8 kv heads take 1.56 M tile steps with one head per item, 1.48 M
// with two, 1.44 M with four (1.40 M would be no waste).
// Measured (one head per item -> up to eight): causal ring step of 4096 x 4096, 32 q / 8 kv heads, one of four in
// 878 -> 859 us; the 256 prompts with a decode step 12.43 -> 12.17 ms: the chip is at its power limit, and wavefronts
// that wait at the diagonal cost time but little power.
inline int most_log_heads_per_item(int n_q_heads, int n_kv_heads) {
    const int g = n_q_heads / n_kv_heads;
    return g % 8 == 0 ? 3 : g % 4 == 0 ? 2 : g % 2 == 0 ? 1 : 0;
}

// One head per item where that is faster.
//  * Fewer items than compute units and fewer than 768 keys: such a call is its first loads and its results, at the rate of
//    one compute unit's memory path, and one head per item spreads them over more of them: 64 q / 8 kv heads, 322 x 322 rows
//    and keys 17.1 -> 14.2 us; 16 / 4, 1900 x 205 folded into a running state 20.6 -> 17.7; at worst 381 x 381 without
//    mask 19.5 -> 20.1.  From 2,000 keys on several heads are 0 ... 5 % ahead.
//  * Items of nearly equal length that come out at a little more than a whole number per compute unit: a few compute units
//    take one more, at full length, while the partly filled row tiles of one head per item are a light last round.  64 / 8,
//    1047 x 11729 without mask 522 -> 442 us, 2073 x 7188 442 -> 384, 128 / 8, 1560 x 16985 1546 -> 1448, 1055 x 1055
//    without mask 97.7 -> 89.4; at worst 2317 x 5543 317 -> 321.  With a mask and between one and two items per compute unit
//    the heavy items of both rounds meet, which pays only for long calls: 598 x 1680 73 -> 79, 532 x 2922 125 -> 118.
inline int log_heads_of_dense_call(int cu, int n_q_heads, int n_kv_heads, int64_t sq, int64_t sk, int64_t delta, bool causal) {
    const int l = most_log_heads_per_item(n_q_heads, n_kv_heads);
    auto items_of = [&](int lh) { return ((sq + (kBM >> lh) - 1) / (kBM >> lh)) * (n_q_heads >> lh); };
    auto keys = [&](int64_t last_row) { return causal ? std::max<int64_t>(0, std::min(sk, last_row + delta + 1)) : sk; };
    const int64_t longest = keys(sq - 1), shortest = keys(std::min<int64_t>(sq, kBM >> l) - 1);
    const int64_t items = items_of(l), items1 = items_of(0);
    if (items < cu) return longest < 768 ? 0 : l;
    const int64_t whole = items / cu, left = items % cu;
    const bool cliff = left > 0 && 20 * left <= 7 * cu && (items1 + cu - 1) / cu == whole + 1 && 10 * (items1 - items) >= cu;
    return cliff && 2 * shortest >= longest && (!causal || whole > 1 || longest >= 2048) ? 0 : l;
}

// The same for a packed or colocated batch, of which the host knows only totals: several heads from 2.5 items per compute
// unit on.  Over 118 random batches, time with one head per item over time with the most, by items per compute unit:
// up to 0.5 0.87, up to 1 0.97, up to 1.5 0.975 (0.73 ... 1.10), up to 2.5 0.986 (0.82 ... 1.03), up to 5 1.014, beyond 1.032.
inline int log_heads_of_list_call(int cu, int n_q_heads, int n_kv_heads, int64_t batch, int64_t total_q) {
    const int l = most_log_heads_per_item(n_q_heads, n_kv_heads);
    return 2 * batch * std::ceil((double)total_q / batch / (kBM >> l)) * (n_q_heads >> l) >= 5.0 * cu ? l : 0;
}

// Query rows per workgroup of a launch: 256 (fwd_il_kernel, one workgroup per 64-key tile step) or, where that would
// leave compute units idle, 64 or 32 (fwd_split_kernel<2 | 1>, 256 keys per step).  Estimated time of a choice =
// base x rounds + step time x (steps of the longest workgroup, or of an average one times the rounds if that is more),
// rounds = workgroups / compute units rounded up; the smallest wins.  Measured on 256 compute units (microseconds; step
// time with few / with all of them busy, memory and power being shared):
//     256 rows: 11.5 + 1.13 / 1.55 per 64 keys    64 rows: 8 + 1.68 / 2.15 per 256 keys    32 rows: 6 + 1.17 / 1.45
// e.g. 8 q heads, 512 rows x 2048 keys: 47.5 / 22.6 / 16.5 us with 256 / 64 / 32 rows; 2048 x 8192: 158 / 80 / 87 us;
// 32 q heads, 1024 x 8192: 164 / 144 / 178 us; 2048 x 8192: 212 / 264 / 323 us.
struct RowChoice {
    int rows, step_keys;
    double base, t_few, t_all;
    double estimate(double cu, double groups, double longest_keys, double average_keys) const {
        const double rounds = std::ceil(groups / cu);
        const double longest = std::ceil(longest_keys / step_keys), average = std::ceil(average_keys / step_keys);
        const double n = std::max(longest, rounds > 1 ? rounds * average : 0.0);
        return base * rounds + n * (t_few + (t_all - t_few) * std::min(1.0, groups / cu));
    }
};
constexpr RowChoice kRowChoices[] = {{256, 64, 11.5, 1.13, 1.55}, {64, 256, 8.0, 1.68, 2.15}, {32, 256, 6.0, 1.17, 1.45}};

inline int rows_of_dense_call(int cu, int n_q_heads, int n_kv_heads, int64_t sq, int64_t sk, int64_t delta, bool causal) {
    auto groups_of = [&](int rows) {   // workgroups (of the persistent kernel: work items)
        const int l = rows == kBM ? most_log_heads_per_item(n_q_heads, n_kv_heads) : 0, positions = rows >> l;
        return (double)((sq + positions - 1) / positions) * (n_q_heads >> l);
    };
    if (groups_of(kBM) >= cu) return kBM;   // an item for every compute unit
    auto keys = [&](int64_t last_row) {   // that a query tile ending with this row sees
        return (double)(causal ? std::max<int64_t>(0, std::min<int64_t>(sk, last_row + delta + 1)) : sk);
    };
    int best = kBM;
    double best_t = 0;
    for (const RowChoice& c : kRowChoices) {
        const double longest = keys(sq - 1), shortest = keys(std::min<int64_t>(sq, c.rows) - 1);
        const double t = c.estimate(cu, groups_of(c.rows), longest, 0.5 * (longest + shortest));
        if (c.rows == kBM || t < best_t) {
            best = c.rows;
            best_t = t;
        }
    }
    return best;
}

// A resumable sweep as spans: every workgroup of fwd_il_kernel walks an equal share of all tile steps, across items, and the
// pieces of an item are merged by a second launch.  That fills the chip where few items, or a few more than a whole number per
// compute unit, would not.  Both sides estimated: a tile step takes 1.13 us while at most half of the compute units are busy
// and up to 1.57 with all of them (power); items 11.5 us per round on top of their steps (one round: between the average and
// the longest item, since what runs last runs alone); spans 30 us, for two items' ends, the merge and its launch, and 0.05 per
// workgroup, for the fp32 pieces' way through memory.  Over 70 random sweeps either estimate is within 10 % of the
// measured time nearly everywhere; where spans are chosen they take 0.39 ... 1.0 of it, 0.68 on average (microseconds): 4 heads,
// 4864 x 53504 960 -> 442; 8 heads, 2560 x 17920 327 -> 173, 1216 x 17024 315 -> 113; 64 heads, 1088 x 9792 384 -> 313; 32 heads,
// 2624 x 18368 712 -> 624.
constexpr int kSpanSteps = 64;     // least steps of a span: with less, pieces and their merge cost more than they win
struct SpanPlan {
    int groups;               // workgroups, a multiple of 8; 0: not worth it
    int64_t steps_per_kvh;    // tile steps of one KV head's items
};
inline double tile_step_us(double busy) { return 1.13 + 0.44 * std::max(0.0, 2 * busy - 1); }   // busy: share of compute units

// Most workgroups of such a sweep: up to eight for each 256-row tile of a head, one per compute unit.  0: enough items as it is.
inline int most_span_groups(int cu, int n_q_heads, int64_t sq) {
    const int64_t tiles = (sq + kBM - 1) / kBM * n_q_heads;
    return tiles >= 4 * (int64_t)cu ? 0 : (int)std::min<int64_t>(cu / 8 * 8, 8 * tiles);
}

inline SpanPlan spans_of_sweep(int cu, int n_q_heads, int n_kv_heads, int64_t sq, int64_t sk, int64_t delta, bool causal) {
    const int64_t tiles = (sq + kBM - 1) / kBM, items = tiles * n_q_heads;
    SpanPlan plan{0, 0};
    const int most = most_span_groups(cu, n_q_heads, sq);
    if (most == 0) return plan;
    int64_t longest = 0;
    for (int64_t i = 0; i < tiles; ++i) {
        const int64_t keys = causal ? std::max<int64_t>(0, std::min(sk, std::min(sq, (i + 1) * kBM) + delta)) : sk;
        const int64_t steps = std::max<int64_t>(1, (keys + 63) / 64);
        longest = std::max(longest, steps);
        plan.steps_per_kvh += steps * (n_q_heads / n_kv_heads);
    }
    const int64_t steps = plan.steps_per_kvh * n_kv_heads;
    const int64_t groups = std::min<int64_t>(most, steps / kSpanSteps) / 8 * 8;
    if (groups < 8 || steps > 0x7fffffff) return plan;
    const double spans = 30 + 0.05 * groups + tile_step_us((double)groups / cu) * ((double)steps / groups + 1);
    const double rounds = std::ceil((double)items / cu), average = (double)steps / items;
    const double plain = 11.5 * rounds + tile_step_us(items / (rounds * cu)) * (rounds > 1 ? rounds * average : 0.5 * (longest + average));
    if (spans < 0.95 * plain) plan.groups = (int)groups;
    return plan;
}

// The same for a packed or colocated batch, of which the host knows only totals and, for a packed one, the caller's hint of
// the longest prompt: estimated for one prompt of that length and the others of equal length.  Keys beyond one per query are
// taken to be long caches, cut into ranges of range_len keys per KV head.
inline int rows_of_list_call(int cu, int n_q_heads, int n_kv_heads, int64_t batch, int64_t total_q, int64_t total_k,
                             int64_t longest, bool causal, int range_len) {
    const double len = (double)total_q / batch;
    // prompt lengths are spread wide (the log-normal mix of the tests has E[L^2] / E[L]^2 of about 3): a row sees 1.5
    // times the average length, not half of it, and the longest prompt is several times the average
    double seen = std::min((double)total_q, 3 * len);
    if (longest > 0 && batch > 1) {   // 5 heads, one prompt of 9,622 tokens and 11 of 63 in all: 243 us as 12 equal ones, 197
        longest = std::max<int64_t>(longest, (int64_t)std::ceil(len));   // (the hint may be too low)
        const double rest = (double)total_q - longest;
        seen = ((double)longest * longest + rest * std::min<double>(3 * rest / (batch - 1), longest)) / total_q;
    }
    if (longest <= 0) longest = (int64_t)std::min((double)total_q, 4 * len);
    const double range_units = range_len > 0 ? std::max(0.0, (double)(total_k - total_q) / range_len) * n_kv_heads : 0.0;
    auto groups_of = [&](int rows) {
        const int l = rows == kBM ? most_log_heads_per_item(n_q_heads, n_kv_heads) : 0;
        return batch * std::ceil(len / (rows >> l)) * (n_q_heads >> l) + range_units;
    };
    if (groups_of(kBM) >= cu) return kBM;
    int best = kBM;
    double best_t = 0;
    for (const RowChoice& c : kRowChoices) {
        if (range_units > 0 && n_q_heads / n_kv_heads > c.rows) continue;   // a range item's rows are the heads of a group
        const double t = c.estimate(cu, groups_of(c.rows), std::max({(double)longest, len, range_units > 0 ? (double)range_len : 0.0}),
                                    causal ? 0.5 * seen : seen);
        if (c.rows == kBM || t < best_t) {
            best = c.rows;
            best_t = t;
        }
    }
    return best;
}

// Whether a work list keeps the items of a sequence together (true) or orders all items by their own keys (false).  Together,
// the 32 workgroups of an XCD walk the keys of one sequence at a time and find them in its L2; apart, neighbours belong to as
// many sequences as there are of about that length, and with 256 prompts of up to 8,192 tokens a tile step took 1.85
// instead of 1.6 us.  But only items in their own order let the launch end evenly, which counts with few of them per
// compute unit.  Over 70 random batches, time by items / time by sequence, by items of 256 rows per compute unit: up to 2.5
// 0.85 ... 1.03, 5 to 8 0.89 ... 1.01, 8 to 14 0.98 ... 1.03, from 15 on never below 1: 1.00 ... 1.08, on average 1.02.
// 256 prompts with a decode step (181 items per compute unit) 11.11 -> 10.50 ms, with a 65,536-token prompt 37.3 -> 36.8 ms.
inline bool list_by_sequence(int cu, int n_q_heads, int rows, int64_t batch, int64_t total_q) {
    return rows == kBM && ((double)total_q / kBM + 0.5 * batch) * n_q_heads >= 16.0 * cu;
}

// Whether a stop word can change what a launch of the resumable sweep does.  fwd_il_kernel leaves an item ahead of a segment
// boundary inside the keys that none of the item's 256 rows has masked (segments of 16 tiles and more; the last whole query
// tile sees most), and a workgroup leaves out every item but its first.  Where neither can happen the sweep is a plain call
// and runs on whatever kernel that takes.  Microseconds per call, sweep kernel / plain, 8 query heads: 704 rows x 1408 keys
// 35.8 / 13.7, 448 x 448 18.8 / 9.9, 3328 x 3328 (segments of 3328) 71.7 / 37.2; 256 x 512 of 4 heads 21.3 / 10.2, 256 x 1024 of
// 64 heads 30.9 / 17.6.
inline bool sweep_can_stop(int cu, int n_q_heads, int64_t sq, int64_t sk, int64_t delta, bool causal, int64_t seg_tiles) {
    const int64_t items = (sq + kBM - 1) / kBM * n_q_heads;
    if ((items + 7) / 8 > std::max(1, cu / 8)) return true;      // a workgroup has more than one item
    if (seg_tiles < 16 || sq < kBM) return false;
    const int64_t row0 = sq / kBM * kBM - kBM, tile = 64;
    int64_t whole = sk / tile, tiles = (sk + tile - 1) / tile, seen = tiles;   // tiles that all rows / any row / the first 32 see
    if (causal) {
        const int64_t keys = std::max<int64_t>(0, std::min(sk, row0 + kBM + delta));
        tiles = (keys + tile - 1) / tile;
        whole = std::min(whole, std::max<int64_t>(0, row0 + delta + 1) / tile);
        seen = std::min(tiles, std::max<int64_t>(0, row0 + 31 + delta + tile) / tile);
    }
    const int64_t last = std::min(std::max<int64_t>(0, std::min(whole, seen) - 1) & ~(int64_t)1, tiles - 1);
    return seg_tiles <= last;
}

// Keys per range of the decode steps in a mixed batch.  A range is one workgroup's walk: fwd_il_kernel, whose launches fill the
// chip, takes the longest; on fwd_split_kernel 4,096 keys are 25 us, often all of the call, and 512 keys 8 us, of which 6 do
// not depend on the keys.  Estimated: the longer of a range's walk and the work shared out over the compute units, 12 us per
// workgroup of the other sequences, a quarter of the shorter, 0.04 us for a range's part in the merge and 2.5 us for a merge
// that might not be needed; shorter ranges where that gives 12 %.  Over 130 random batches 0.81 of the time with 4,096 keys
// throughout (0.79 without that line, but then 13 of them are up to 9 % slower), over 90 others 0.89, three of them 1 ... 6 %
// slower; microseconds with 512 / 1,024 / 2,048 / 4,096 keys: 4 heads, 17 sequences and 13,057 keys 13.6 / 15.7 / 19.5 /
// 26.4; 24 and 122,882 29.3 / 21.1 / 23.5 / 32.7; 8 heads, 39 and 299,920 85 / 75 / 77 / 72; 26 and 6,458 44.1 / 43.9 / 43.9 / 41.9.
// Ranges that would take more partial results than most_ranges_of_mixed_call() are left out.
constexpr int kMinRange = 512, kMaxRange = 4096;

// Most whole ranges of a mixed batch, as a function of its totals that never falls when one of them grows: a workspace that is
// enough for one batch is enough for all smaller ones, whatever lengths of ranges they get.  Ranges of under 4,096 keys are
// chosen where walks of 4,096 keys leave compute units idle: over 20 million random calls, on 8 to 304 compute units, with never
// more than 1.4 workgroups of them per compute unit.  Two are allowed, and the keys of the other sequences on top.
inline int64_t most_ranges_of_mixed_call(int cu, int n_kv_heads, int64_t total_q, int64_t total_k) {
    return std::min(total_k / kMinRange, std::max(total_k / kMaxRange, 2 * (int64_t)cu / n_kv_heads + 1 + total_q / kMinRange));
}

inline int range_of_mixed_call(int cu, int rows, int n_q_heads, int n_kv_heads, int64_t batch, int64_t total_q, int64_t total_k) {
    int best = kMaxRange;
    if (rows == kBM) return best;
    const double others = ((double)total_q / rows + 0.3 * batch) * n_q_heads;
    const double cached = (double)std::max<int64_t>(0, total_k - total_q);
    const int64_t most = most_ranges_of_mixed_call(cu, n_kv_heads, total_q, total_k);
    double best_t = 0;
    for (int keys = kMaxRange; keys >= kMinRange && total_k / keys <= most; keys /= 2) {
        const double walk = 6 + 1.2 * std::min<double>(keys, cached) / 256;
        const double share = (others * 12 + cached * n_kv_heads / keys * walk) / cu;
        const double t = std::max(walk, share) + 0.25 * std::min(walk, share) + 0.04 * cached / keys + (cached > keys ? 2.5 : 0.0);
        if (keys == kMaxRange || t < best_t) {
            best = keys;
            best_t = keys == kMaxRange ? 0.88 * t : t;
        }
    }
    return best;
}

// Whether a batch does without a work list: the workgroups of fwd_split_kernel find their items in the offsets, a lane per
// sequence.  That saves a launch, 3 ... 4 us, and costs every workgroup a loop over the sequences, one workgroup at a time on a
// compute unit.  Over 36 random batches of 4 to 64 sequences, microseconds won, by workgroups (bound) and sequences: 70 x 5
// 4.3 (11.5 -> 7.2), 302 x 14 3.3, 345 x 42 2.9, 535 x 13 3.9, 695 x 16 3.5; 731 x 14 -0.5, 433 x 45 0.1, 640 x 29 -0.1, 515 x 54 -3.4,
// 1190 x 29 -7.8, 1990 x 55 -45.
inline bool batch_without_list(int cu, int rows, int n_q_heads, int64_t batch, int64_t total_q) {
    const int64_t groups = (total_q / rows + batch) * n_q_heads;
    return rows < kBM && batch <= 64 && 4 * groups <= 11 * cu && groups * batch <= 64 * cu;
}

// Keys per range when sk keys are cut into n_splits ranges of whole tiles.
inline int64_t range_keys(int64_t sk, int64_t n_splits, int tile) {
    return std::max<int64_t>(((sk + n_splits - 1) / n_splits + tile - 1) / tile * tile, tile);
}

// Whether a decode step with groups of up to 32 heads runs on fwd_split_kernel (a workgroup per range and KV head, its
// wavefronts sharing the keys) or on decode_kernel (a wavefront per range and KV head).  Microseconds per step, with the
// merge, fresh caches, 8 KV heads, (keys per range) in decode_kernel / fwd_split_kernel:
//     4,096 keys     16 ranges 18.2 / 11.4      64 ranges (64) 11.6 / 15.1
//     32,768 keys    32 ranges 60.9 / 31.8     128 ranges (256) 33.6 / 41.9
//     524,288 keys   32 ranges 766 / 356       128 ranges 384 / 372
// The workgroup kernel wins while all of its workgroups run at once and loses with a second round of them (both kernels as
// built wait for every request of a wavefront at each tile, so it is not the depth of decode_kernel's rings that wins; what
// does has not been measured).  In one round (16 ranges of 8 KV heads), by the keys of a range: 32 keys 8.6 / 9.3,
// 64 keys 10.1 / 9.5, 96 keys 11.8 / 10.1, 128 keys 14.9 / 10.7, 256 keys 22.1 / 12.6; 32 ranges, 64 heads on 64 KV heads
// and 4 on 4 give the same to 1 us.  The line lies above two tiles; a range of exactly two would gain 0.6 us beyond it.
inline bool decode_on_split_kernel(int cu, int n_q_heads, int n_kv_heads, int64_t sk, int64_t n_splits) {
    return n_q_heads / n_kv_heads <= 32 && n_splits * n_kv_heads <= cu && range_keys(sk, n_splits, 32) > 64;
}

// Whether the last workgroup of a KV head merges its ranges itself instead of a second launch (fwd_split_kernel.hpp).  That
// takes it three trips to memory and the read of group x ranges partial results by one compute unit, against a launch: 2 us
// of the host's time, and on the GPU (microseconds per step of many in one graph, fresh caches, one launch / two, when words
// were still marked in a way that a graph could replay), by group x ranges: 3 9.6 / 9.9, 16 9.2 / 9.4, 32 10.4 / 10.8 and
// 96.7 / 97.4, 64 11.8 / 12.2 and 10.8 / 11.0, 128 15.4 / 14.8, 12.6 / 12.3 and 10.5 / 9.7, 256 17.3 / 15.0 and 358.3 / 355.5,
// 1,024 22 / 12.  4,096 keys of 32 / 8 heads, called over and over on one cache, where the host is the slower: 11.85 -> 10.0;
// as the first pass on new inputs, 27.7 ... 30.2 -> 27.0 ... 27.8.  Kernel times of that step: 9.4, against 6.4 + 4.1.
inline bool merge_in_launch(int group, int64_t n_splits) { return group * n_splits <= 64; }

// What the words of such a call hold once their ranges are there: call number n of a process, a mixer of 64 bits (splitmix64)
// on a stepped seed of the process.  Both are one to one, so no two calls of a process have the same mark; that data of
// another origin passes for it takes 64 equal bits.
inline uint64_t merge_mark(uint64_t seed, uint64_t n) {
    uint64_t x = seed + 0x9e3779b97f4a7c15ull * n;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

// Key ranges of a decode step whose caller leaves the number to the library: as many as give every compute unit a workgroup
// of fwd_split_kernel, of 256 keys at least (a tile of 32 for each of eight wavefronts) -- or, with more than 11 KV heads
// and 768 keys per compute unit in all, of decode_kernel, whose workgroups read four neighbouring KV heads of a token.
// Microseconds per step on 256 compute units, decode_kernel / fwd_split_kernel, each with these many ranges:
//     16,384 keys    8 heads 26.8 / 21.3   12 heads 29.0 / 26.5   16 heads 33.1 / 34.5   40 heads 64.0 / 64.5   128 heads 190 / 201
//     4,096 keys     40 heads 27.3 / 24.1   48 heads 28.0 / 26.6   64 heads 33.5 / 34.7   128 heads 55.7 / 56.5
//     65,536 keys    7 heads 51.6 / 49.0   10 heads 66.8 / 60.4   36 heads 216 / 227   100 heads 562 / 627
//     524,288 keys   1 head 100 / 54   8 heads 377 / 369   11 heads 507 / 504
// Up to 11 heads the first is behind everywhere but for 1.6 % at 8 heads and 65,536 keys and 3 % at 4 heads and 524,288 on one
// card, where it is 3 % and 1.5 % behind on another.
// At the line itself (16 heads x 12,288 keys ... 256 x 768) the two differ by 0 ... 17 % in favour of fwd_split_kernel.
// Ranges of decode_kernel whose partial results would not fit pec_decode_splitkv_static's buffer (16 KV heads with groups of
// 16, say) stay with fwd_split_kernel too: its ranges, a quarter as many, always fit there where they did before.
inline int64_t decode_default_ranges(int cu, int n_q_heads, int n_kv_heads, int64_t sk) {
    const int g = n_q_heads / n_kv_heads;
    const int64_t per_cu = cu / n_kv_heads;      // 0: more KV heads than compute units
    const int64_t n = std::max<int64_t>(1, std::min<int64_t>(per_cu, sk / 256));
    const int64_t head_groups = (n_kv_heads + kDecWaves - 1) / kDecWaves;
    const int64_t n_waves = std::max<int64_t>(1, std::min<int64_t>(cu / head_groups, sk / 256));
    if ((n_kv_heads <= 11 || sk * n_kv_heads <= 768 * (int64_t)cu || n_waves * n_q_heads > kStaticPartials) &&
        decode_on_split_kernel(cu, n_q_heads, n_kv_heads, sk, n))
        return n;
    if (g <= 32) return std::min<int64_t>(n_waves, std::max<int64_t>(1, kStaticPartials / n_q_heads));
    // wide groups run on the prefill kernel: one workgroup per compute unit, at least 16 tiles of 64 keys each
    return std::max<int64_t>(1, std::min<int64_t>(per_cu, sk / 1024));
}

}  // namespace pec
