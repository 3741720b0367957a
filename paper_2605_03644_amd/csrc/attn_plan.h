// How attention calls are cut into workgroups: which kernel a call runs, its row blocks and its context splits.  Host logic
// over sizes alone -- no HIP types here, so that it can be compiled and checked without a GPU.
#pragma once
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <functional>
#include <utility>
#include <vector>

#include "adapshot.h"

namespace adapshot {

constexpr int kAttnRowTile = 256;  // query rows per workgroup of the MFMA kernel
// With at most this many rows per kv head half of a workgroup's wavefronts only move tiles and the launch is bound
// by the memory path, not by the matrix cores: its tile loads are then marked non-temporal (when no other workgroup
// reads the same tiles).
constexpr int kAttnStreamRows = 128;
// ---- streaming attention (attn_stream_kernel.h)
constexpr int kStreamWaves = 8;       // wavefronts per workgroup, each with keys of its own
constexpr int kStreamItems = 32;      // attention problems per launch (their descriptions travel in the kernel arguments)
constexpr int kStreamMaxSplits = 64;  // context splits per problem
constexpr int kStreamUnits = 4096;    // (problem, row tile, kv head) units of a launch that is split: one arrival counter each
// Distance of the arrival counters of n units (of an entropy call: rows), in counters: up to a 128-byte line each.  Atomics
// on one line follow each other at about 14 ns whatever counter they name (16 rows x 126 arrivals in one line: 29 us, a line
// for every row: 10 us).
inline int32_t counter_stride(int64_t n) {
    return (int32_t)(n >= kStreamUnits ? 1 : kStreamUnits / n < 32 ? kStreamUnits / n : 32);
}

// The tile kernel's shapes (attn_mfma.hip).
inline bool attn_mfma_supported(const adapshot_model_desc& d) { return d.dtype == ADAPSHOT_BF16 && d.head_dim == 128; }

// Split count of one MFMA attention launch.  The grid is `units` (kv head, row tile) pairs times the context
// splits, plus one workgroup per unit for the query's own tokens; one workgroup occupies a compute unit, and
// the self workgroups are dispatched first.  A handful of candidate counts -- everything in one round beside
// the self workgroups, one context split per compute unit with the last of them starting when the self
// workgroups are done, and two to four rounds of that -- are priced in 64-key tiles plus a fixed
// per-workgroup cost, and the cheapest wins (the smaller count on a tie).  A short context fits everything into
// one round (26k tokens, 16 units: 15 splits of 29 tiles beside the 16 self workgroups); a long one does not
// leave the self workgroups' compute units idle (127k tokens, 64 units: 4 splits of 495 tiles, not 3 of 660).
inline int64_t plan_mfma_splits(int64_t n_cu, int64_t units, int64_t key_tiles, int64_t self_tiles) {
    const double fixed = 2.5;  // launch, first tile round trip and partial write-out of a workgroup, in tiles
    const int64_t s_max = std::min<int64_t>(key_tiles, 64);
    const double ls = (double)self_tiles + fixed;
    auto price = [&](int64_t s) {
        const double l = (double)((key_tiles + s - 1) / s) + fixed;
        const int64_t n = units * s;
        double t;
        if (units + n <= n_cu) t = std::max(l, ls);          // one round
        else if (n <= n_cu && units <= n_cu) t = ls + l;      // the context workgroups that do not fit wait for the self ones
        else t = ceil(((double)n * l + (double)units * ls) / ((double)n_cu * l)) * l;  // whole rounds
        return t + 0.02 * (double)s;                           // partials cost a little too
    };
    const int64_t one_round = (n_cu - units) / units, per_cu = n_cu / units;
    const int64_t cand[6] = {1, one_round, per_cu, 2 * per_cu, 3 * per_cu, 4 * per_cu};
    int64_t best = 1;
    double best_t = price(1);
    for (int64_t c : cand) {
        int64_t sc = std::max<int64_t>(1, std::min<int64_t>(c, s_max));
        sc = (key_tiles + ((key_tiles + sc - 1) / sc) - 1) / ((key_tiles + sc - 1) / sc);  // the count this split length gives
        const double t = price(sc);
        if (t < best_t - 1e-9 || (t < best_t + 1e-9 && sc < best)) {
            best = sc;
            best_t = t;
        }
    }
    return best;
}

// 16-row blocks per workgroup of the streaming kernel.  Two share the loads of K and V, but leave half the workgroups: fp32
// models want two workgroups per compute unit with one block each before that pays, bf16 models, whose products cost
// less, half a workgroup and a context of some length (64 query tokens of 32/8 heads, one block / two: 6.4k slots
// 43.6 / 38.3 us, 2.3k 27.8 / 27.6, 742 20.0 / 22.6; 32 tokens, 6.4k slots 34.0 / 34.1).  And the second blocks have to hold
// rows, at least half of them: problems share no workgroup (32 queries of 16 rows over 2k / 4k slots: two blocks, the second
// one empty, 27.2 / 49.8 us, one 24.8 / 47.3).
struct StreamShape {
    int64_t rows, key_tiles;  // query rows per kv head, 64-key tiles of context
};
inline int32_t stream_row_blocks(const adapshot_model_desc& d, int64_t n_cu, const StreamShape* shapes, int32_t n_shapes) {
    if (d.head_dim != 64) return 1;
    int64_t blocks = 0, pairs = 0, key_tiles = 0;
    for (int32_t i = 0; i < n_shapes; ++i) {
        blocks += (shapes[i].rows + 15) / 16;
        pairs += (shapes[i].rows + 31) / 32;
        key_tiles = std::max(key_tiles, shapes[i].key_tiles);
    }
    if (4 * pairs > 3 * blocks) return 1;
    blocks *= d.n_kv_heads;
    return blocks >= 2 * n_cu || (d.dtype == ADAPSHOT_BF16 && 2 * blocks >= n_cu && key_tiles >= 32) ? 2 : 1;
}
// (problem, row tile, kv head) units of a problem
inline int64_t stream_units(const adapshot_model_desc& d, const StreamShape& s, int32_t row_blocks) {
    return d.n_kv_heads * ((s.rows + 16 * row_blocks - 1) / (16 * row_blocks));
}

// Keys of a step of one wavefront.
inline int64_t stream_step_keys(const adapshot_model_desc& d) { return d.dtype == ADAPSHOT_BF16 && d.head_dim <= 128 ? 32 : 16; }
// Splits of a problem whose context is cut into pieces of split_tiles 64-key tiles; the last one also takes the query's own tokens.  (A
// split of their own, where these give the last one's wavefronts another step, is one more partial and gained nothing: 1357 calls
// and batches within 0.5 % either way.)
inline int64_t stream_splits(const StreamShape& s, int64_t split_tiles) {
    return std::max<int64_t>(1, (s.key_tiles + split_tiles - 1) / split_tiles);
}

// What a launch of the streaming kernel takes, us, by its longest split (in 64-key tiles).  A workgroup has a compute unit to itself and
// spends 3.4 us before its first product and after its last one, and on every step of its wavefronts 0.25 us plus the loads of 54 KB/us
// (where the steps do not divide by the wavefronts, some of these run one step fewer: the others get more of the memory then).
// As many workgroups as there are compute units run at once, the next ones after them, and each turn takes at least what the memory needs
// for its share of the keys: 2.4 TB/s to 64 workgroups, 3.4 to 128, 6.1 to 256; rows of one kv head in several units are drawn
// from it half of the time.  Splits cost their merge by the last workgroup: 3.2 us, 0.15 for every round of its loads and 19 ns per KB.
// Fitted to 1294 calls over contexts that no cache held, each with up to 20 split counts (single calls of 11 models, 1 to 256 tokens over
// 60 to 32k slots; decode steps of 2 to 32 queries of 5 models), with a merge that took splits one branch at a time: the counts chosen took 0.8 %
// longer than the best ones.  The merge has become shorter since and the price has not: over 107 such calls of 8 models the counts chosen take
// 6.1 % longer, at most 25 % (64/8 heads x 128, 8 tokens over 330 slots 7.9 us, in one split 6.3; 28/4 heads, one over 16k, 42 splits 12.5 to 12.8, 51 and 63 12.4).
inline double stream_price(const adapshot_model_desc& d, int64_t n_cu, const StreamShape* shapes, int32_t n_shapes, int32_t row_blocks,
                           int64_t split_tiles) {
    const int64_t e = d.dtype == ADAPSHOT_BF16 ? 2 : 4, sk = stream_step_keys(d);
    int64_t wgs = 0, read = 0, drawn = 0, longest = 0, rows = 0;  // tiles of a kv head: read by all workgroups, by one unit of each problem
    for (int32_t i = 0; i < n_shapes; ++i) {
        const int64_t here = stream_units(d, shapes[i], row_blocks);
        wgs += here * stream_splits(shapes[i], split_tiles);
        read += here * shapes[i].key_tiles;
        drawn += d.n_kv_heads * shapes[i].key_tiles;
        longest = std::max(longest, shapes[i].key_tiles);
        rows = std::max(rows, std::min<int64_t>(shapes[i].rows, 16 * row_blocks));
    }
    const int64_t steps = std::min(split_tiles, longest) * 64 / sk, step_rounds = (steps + kStreamWaves - 1) / kStreamWaves;
    const double round_us = 0.25 + (double)(kStreamWaves * sk * 2 * d.head_dim * e) * (row_blocks == 2 ? 1.41 : 1.0) / 54e3;
    const double wg_us = 3.4 + (0.4 * (double)step_rounds + 0.6 * (double)steps / kStreamWaves) * round_us;
    const double mb_per_wg = 0.5 * (double)((read + drawn) * 128 * d.head_dim * e) * 1e-6 / (double)wgs;
    auto turn = [&](double n) { return std::max(wg_us, 3.4 + mb_per_wg * (n + 250.0) / 12.0); };
    double t = (double)(wgs / n_cu) * turn((double)n_cu) + (wgs % n_cu > 0 ? turn((double)(wgs % n_cu)) : 0.0);
    if (split_tiles < longest) {
        const int64_t n = (longest + split_tiles - 1) / split_tiles;
        const int64_t pieces = std::max<int64_t>(1, rows * d.head_dim / 4), threads = 64 * kStreamWaves;
        const int64_t groups = std::max<int64_t>(1, std::min(threads / pieces, (n + 7) / 8));
        const int64_t loads = ((pieces + threads / groups - 1) / (threads / groups)) * ((n + 8 * groups - 1) / (8 * groups));
        t += 3.2 + 0.15 * (double)loads + 0.019 * (double)(n * rows * d.head_dim * 4) / 1024.0;
    }
    return t;
}

// Split length (in 64-key tiles) of a launch: the longest context in n equal splits, the others in splits of the same length.
inline int64_t plan_stream_split_tiles(const adapshot_model_desc& d, int64_t n_cu, const StreamShape* shapes, int32_t n_shapes,
                                       int32_t row_blocks) {
    int64_t longest = 0, units = 0;
    for (int32_t i = 0; i < n_shapes; ++i) {
        longest = std::max(longest, shapes[i].key_tiles);
        units += stream_units(d, shapes[i], row_blocks);
    }
    if (longest == 0) return 1;
    // (beyond two turns nothing is gained, and the host has better things to do)
    const int64_t n_max = std::min<int64_t>(std::min<int64_t>(longest, kStreamMaxSplits), 2 * n_cu / std::max<int64_t>(units, 1) + 1);
    int64_t best = longest, last = 0;
    double best_t = 1e300;
    for (int64_t n = 1; n <= n_max; ++n) {
        const int64_t st = (longest + n - 1) / n;
        if (st == last) continue;  // no shorter splits than with one fewer
        last = st;
        const double t = stream_price(d, n_cu, shapes, n_shapes, row_blocks, st);
        if (t < best_t) {
            best_t = t;
            best = st;
        }
    }
    return best;
}

// One launch of the streaming kernel.  More units than arrival counters: the chip is full without splits, and none are made.
struct StreamPlan {
    int32_t row_blocks;
    int64_t units;        // of all problems
    int64_t split_tiles;  // 64-key tiles of a split
    int64_t n_split;      // of the longest problem (an empty one: 1)
};
inline StreamPlan plan_stream(const adapshot_model_desc& d, int64_t n_cu, int32_t force_splits, const StreamShape* shapes,
                              int32_t n_shapes) {
    StreamPlan p;
    p.row_blocks = stream_row_blocks(d, n_cu, shapes, n_shapes);
    p.units = 0;
    int64_t tiles = 1;
    for (int32_t i = 0; i < n_shapes; ++i) {
        p.units += stream_units(d, shapes[i], p.row_blocks);
        tiles = std::max(tiles, shapes[i].key_tiles);
    }
    if (p.units > kStreamUnits) p.split_tiles = tiles;
    else if (force_splits > 0) p.split_tiles = (tiles + force_splits - 1) / force_splits;
    else p.split_tiles = plan_stream_split_tiles(d, n_cu, shapes, n_shapes, p.row_blocks);
    p.split_tiles = std::max(p.split_tiles, (tiles + kStreamMaxSplits - 1) / kStreamMaxSplits);
    p.n_split = (tiles + p.split_tiles - 1) / p.split_tiles;
    return p;
}

// Which kernel: the 256-row tile kernel for bf16 models of head dimension 128 where it is the cheaper one.  It reads a context
// once per 256 rows and draws 6.1 TB/s, but is two launches (a batch whose tables do not fit the kernel arguments: three), leaves wavefronts
// without rows idle and writes a partial for every split; the streaming kernel reads it once per 16 rows, in one launch.
constexpr int64_t kStreamBytes = 200000000;
inline int64_t context_bytes(const adapshot_model_desc& d, int64_t slots) { return slots * d.n_kv_heads * d.head_dim * 4; }

// A single call compares prices, but keeps the streaming kernel's fp32 partials where it has few rows.  The tile kernel's price: 10.8 us
// for the two launches, 0.83 us per MB of partials, 0.08 per split, and per tile of a workgroup and turn 0.35 or (more than 128 rows)
// 0.57 us, or 7.3 MB/us.  Fitted to 358 calls (5 models, 1 to 256 tokens over 60 to 32k slots that no cache held); the streaming kernel's merge has become
// shorter since: over 121 such calls the kernel chosen is 1.5 % slower than the better one, at most 39 % (8/2 heads, 58 tokens over 12k 25.5 by
// tiles, 18.3 by streaming; 28/4 heads, 76 over 1.8k 20.0 and 14.5).  Us a call, call after call, tile kernel / streaming: 32/8 heads, 8 tokens over
// 250 / 2k / 4k slots 11.4 / 15.3 / 16.7 and 6.2 / 9.0 / 10.4; 32 tokens over 1k / 4k 15.8 / 19.5 and 9.6 / 17.4; 64 tokens over 250 / 1k / 4k
// 14.2 / 18.0 / 23.5 and 7.4 / 11.2 / 24.5; 28/4 heads, 16 / 64 tokens over 4k 21.6 / 22.3 and 12.5 / 23.1; 64/8 heads, 8 tokens over 8k 20.0 and 19.3.
inline bool single_by_tiles(const adapshot_model_desc& d, int32_t t_q, int64_t n_ctx, bool zero_copy, int64_t n_cu = 256) {
    if (!attn_mfma_supported(d)) return false;
    if (zero_copy || context_bytes(d, n_ctx) > kStreamBytes) return true;  // (no gathered form of the streaming kernel for these models)
    const int64_t rows = (int64_t)t_q * (d.n_q_heads / d.n_kv_heads), key_tiles = (n_ctx + 63) / 64, self_tiles = ((int64_t)t_q + 63) / 64;
    if (rows <= 8 || (rows <= 16 && n_ctx <= 1024)) return false;
    if (rows > 16 * kAttnRowTile) return true;
    const StreamShape sh{rows, key_tiles + self_tiles};  // (the query's own tokens as more context)
    const int32_t rb = stream_row_blocks(d, n_cu, &sh, 1);
    const double stream = stream_price(d, n_cu, &sh, 1, rb, plan_stream_split_tiles(d, n_cu, &sh, 1, rb));
    const int64_t units = d.n_kv_heads * ((rows + kAttnRowTile - 1) / kAttnRowTile);
    const int64_t n_split = key_tiles > 0 ? plan_mfma_splits(n_cu, units, key_tiles, self_tiles) : 0;
    const int64_t per_wg = n_split > 0 ? (key_tiles + n_split - 1) / n_split : 0, turns = (units * (n_split + 1) + n_cu - 1) / n_cu;
    const double drawn_mb = (double)context_bytes(d, 64 * key_tiles) * 1e-6;
    const double partials_mb = (double)((n_split + 1) * rows * d.n_kv_heads * d.head_dim * 2) * 1e-6;
    return 10.8 + 0.83 * partials_mb + 0.08 * (double)n_split +
               std::max((rows > 128 ? 0.57 : 0.35) * (double)(per_wg * turns), drawn_mb / 7.3) < stream;
}

// A batch of these models: the streaming kernel if every item has at most 16 rows per kv head, all contexts together at most 1.5 times
// kStreamBytes, and every context is read by one item -- items that share one find its tiles in the L2 when the tile kernel orders
// them by cache and split.  Per layer of a decode step over contexts that no cache held, planned anew in every call (tile kernel, its tables in the
// kernel arguments, and merge / streaming kernel, us): 28/4 heads, 16 queries of 4k slots 131 MB 33.1 / 29.1, 12 of 8k 197 MB 44.2 / 40.4, 30 of 4k 246 MB
// 53.7 / 49.9, 8 of 16k 262 MB 50.9 / 53.0, 20 of 8k 328 MB 65.5 / 62.5, 12 of 16k 393 MB 74.8 / 73.9, 16 of 16k 524 MB 96.6 / 97.3; 32/8 heads,
// 4 tokens, 8 of 8k 262 MB 54.3 / 52.8, 12 of 8k 393 MB 76.2 / 78.4, 6 of 16k 393 MB 74.3 / 74.3.  With tables (33 queries of 28/4 heads): of 4k
// 270 MB 70.3 / 60.5, of 8k 541 MB 116.1 / 106.1.  A batch of one takes it where a single call does, too.
inline bool batch_by_stream(const adapshot_model_desc& d, const adapshot_attn_item* items, int32_t n_items, int64_t n_cu) {
    if (!attn_mfma_supported(d)) return true;
    if (n_items == 1 && !single_by_tiles(d, items[0].t_q, items[0].n_ctx, false, n_cu)) return true;
    std::vector<int32_t> seen;
    seen.reserve((size_t)n_items);
    int64_t slots = 0;
    for (int32_t i = 0; i < n_items; ++i) {
        slots += items[i].n_ctx;
        if ((int64_t)items[i].t_q * (d.n_q_heads / d.n_kv_heads) > 16) return false;
        if (context_bytes(d, slots) > (n_items == 1 ? kStreamBytes : kStreamBytes + kStreamBytes / 2)) return false;
        if (items[i].n_ctx > 0) seen.push_back(items[i].cache_index);
    }
    std::sort(seen.begin(), seen.end());
    return std::adjacent_find(seen.begin(), seen.end()) == seen.end();
}

// Split the context of one attention call so that (kv heads x row tiles x splits) fills the chip.  Keys per
// split is a multiple of the 64-key tile; an empty context has no split.  (A zero-copy query of 32/8 heads and one token
// over 26k slots: 30 splits of 14 tiles 35.7 us, 21 of 20, as the streaming kernel would want them, 43.8 us.)
inline void plan_single_attn(const adapshot_model_desc& d, int64_t n_cu, int32_t force_splits, int32_t t_q, int64_t n_ctx,
                             bool zero_copy, int64_t* n_split_out, int64_t* keys_per_split_out) {
    const int64_t rows = (int64_t)t_q * (d.n_q_heads / d.n_kv_heads);
    const int64_t key_tiles = (n_ctx + 63) / 64;
    int64_t n_split = 0, keys_per_split = 64;
    if (key_tiles > 0) {
        if (single_by_tiles(d, t_q, n_ctx, zero_copy, n_cu)) {
            const int64_t units = d.n_kv_heads * ((rows + kAttnRowTile - 1) / kAttnRowTile);
            n_split = force_splits > 0 ? std::min<int64_t>(force_splits, key_tiles)
                                       : plan_mfma_splits(n_cu, units, key_tiles, ((int64_t)t_q + 63) / 64);
            keys_per_split = ((key_tiles + n_split - 1) / n_split) * 64;
        } else {
            const StreamShape sh{rows, key_tiles};
            keys_per_split = plan_stream(d, n_cu, force_splits, &sh, 1).split_tiles * 64;
        }
        n_split = (n_ctx + keys_per_split - 1) / keys_per_split;
    }
    *n_split_out = n_split;
    *keys_per_split_out = keys_per_split;
}

// Common split length (in 64-key tiles) of a batch.  The longest item is cut into n equal splits, every other item
// into splits of that length plus a remainder; n is the candidate whose work list finishes first when the
// workgroups, sorted longest first, are dealt round-robin over the compute units (the first workgroup of every
// round is the longest of that round, so the finish time is the sum of those), or rather the fewest splits that come
// within 12 % of it: whole rounds of equal workgroups win
// over an average that leaves a few compute units one workgroup more (32 queries x 4 kv heads x 16k tokens: 4 splits,
// 512 workgroups in two rounds, 199 us; the 4-or-5 splits of an average-based length: 210 us; 3 splits: 230 us).
struct BatchShape {
    int64_t units, key_tiles, self_tiles;
};
inline int64_t plan_batch_split_tiles(int64_t n_cu, const std::vector<BatchShape>& shapes, int32_t force_splits) {
    int64_t longest = 1;
    for (const BatchShape& b : shapes) longest = std::max(longest, b.key_tiles);
    if (force_splits > 0) return (longest + force_splits - 1) / force_splits;
    const double fixed = 2.5;  // launch, first tile round trip and partial write-out of a workgroup, in tiles
    struct Class {
        double cost;
        int64_t count;
    };
    std::vector<Class> cls;
    int64_t best_st = longest;
    double best_t = 1e300;
    static const int kCand[] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16, 20, 24, 32, 48, 64};
    int64_t cand_st[sizeof(kCand) / sizeof(kCand[0])];
    double cand_t[sizeof(kCand) / sizeof(kCand[0])];
    int n_cand = 0;
    int64_t last_st = -1;
    for (int n : kCand) {
        int64_t st = (longest + n - 1) / n;
        if (st < 8 && longest >= 8) st = 8;  // shorter splits are all prologue
        if (st == last_st) continue;
        last_st = st;
        cls.clear();
        int64_t partials = 0;
        for (const BatchShape& b : shapes) {
            const int64_t full = b.key_tiles / st, rem = b.key_tiles - full * st;
            if (full > 0) cls.push_back(Class{(double)st + fixed, full * b.units});
            if (rem > 0) cls.push_back(Class{(double)rem + fixed, b.units});
            cls.push_back(Class{(double)b.self_tiles + fixed, b.units});
            partials += (full + (rem > 0)) * b.units;
        }
        std::sort(cls.begin(), cls.end(), [](const Class& a, const Class& b) { return a.cost > b.cost; });
        // finish time of the compute unit that gets the first workgroup of every round
        double t = 0.0;
        int64_t rank = 0, next_pick = 0;  // workgroups dealt so far; rank of the next round's first workgroup
        for (const Class& c : cls) {
            while (next_pick < rank + c.count) {
                t += c.cost;
                next_pick += n_cu;
            }
            rank += c.count;
        }
        t += 0.0005 * (double)partials;  // the partials are written and merged too
        cand_st[n_cand] = st;
        cand_t[n_cand++] = t;
        best_t = std::min(best_t, t);
    }
    // The fewest splits within 12 % of the best: the chip clocks higher while some compute units idle, so a finer
    // cut gains less than its balance promises, and every extra workgroup has a prologue, an epilogue and a
    // partial of its own (the probe sweep's 48 items: 4-5 splits of the longest item 850 us, 8-16 splits 872-887 us).
    for (int i = 0; i < n_cand; ++i)
        if (cand_t[i] <= 1.12 * best_t) return cand_st[i];
    return best_st;
}

// The same where the items do not stream their contexts (kAttnStreamRows): items differ in length by design (nested
// prefixes), and equal splits of the longest one fit the others badly.  Candidates are also the lengths that give every
// compute unit k workgroups of equal work, with some slack for the remainders; each is dealt out the way the hardware does it
// (longest first, to the compute unit that is free first) and priced as that finish time plus 0.13 tiles per workgroup.
// That price is fitted to the two rounds of one probe sweep (8 queries; split length: time per layer): prefixes of 128-512
// shots 859: 1120 us, 430: 780, 375: 750, 193: 763, 94: 780, 61: 806; prefixes of 16-64 shots 110: 170 us, 56: 124, 50: 128, 28:
// 137, 8: 190.  (The chip clocks lower the fewer compute units idle, so a better balance gives about half of what it
// promises, which the price per workgroup accounts for.)  Away from that sweep (equal splits / these): 8 queries, 5 nested
// prefixes of 25k tokens, 32/8 heads, 8 / 16 / 33 tokens over caches 253 / 215, 261 / 225, 335 / 309 us, over the pool 360 / 308,
// 368 / 317, 415 / 365, 28/4 heads, 8 tokens 137 / 123 and 192 / 168; zero-copy decode of 32 contexts of 16k slots 208 / 205.  Only
// from 32 tiles per compute unit on: below that a launch is mostly prologues, and the equal splits lose less (2 queries,
// prefixes of 11-91 shots, 13 tiles: a pass of 150 us against 172; 1 query, prefixes of 27-221, 16 tiles: 204 against 228).
//
// Compute units that are free at the same time are dealt to together, so that a plan costs the host what the batch has
// in distinct workgroups, not in workgroups (24 / 64 / 256 items of 7 KV heads: 33 / 157 / 471 us; one workgroup after the other
// 329 / 842 / 2067; equal splits 16 / 53 / 385).
constexpr int64_t kBalancedTiles = 32;
inline int64_t plan_balanced_split_tiles(int64_t n_cu, const std::vector<BatchShape>& shapes) {
    const int64_t fixed2 = 5;  // half tiles: 2.5 tiles of launch, first tile round trip and partial write-out of a workgroup
    const double per_wg = 0.13;
    int64_t longest = 1, total = 0;
    for (const BatchShape& b : shapes) {
        longest = std::max(longest, b.key_tiles);
        total += b.units * b.key_tiles;
    }
    if (total < kBalancedTiles * n_cu) return plan_batch_split_tiles(n_cu, shapes, 0);
    const int64_t floor_tiles = std::min<int64_t>(8, longest);  // shorter splits are all prologue
    std::vector<int64_t> cand;
    for (int n : {1, 2, 3, 4, 6, 8}) cand.push_back((longest + n - 1) / n);
    for (int k : {1, 2, 3, 4})
        for (double f : {1.02, 1.05, 1.1}) cand.push_back((int64_t)ceil((double)total * f / (double)(k * n_cu)));
    for (int64_t& st : cand) st = std::min(longest, std::max(floor_tiles, st));
    std::sort(cand.begin(), cand.end(), std::greater<int64_t>());
    cand.erase(std::unique(cand.begin(), cand.end()), cand.end());
    typedef std::pair<int64_t, int64_t> Class;  // (cost in half tiles, workgroups); of compute units: (time they are free, how many)
    std::vector<Class> cls, level;
    int64_t best_st = longest;
    double best_t = 1e300;
    for (int64_t st : cand) {
        cls.clear();
        int64_t n_full = 0, n_wg = 0;
        for (const BatchShape& b : shapes) {
            const int64_t full = b.key_tiles / st, rem = b.key_tiles - full * st;
            n_full += full * b.units;
            if (rem > 0) cls.push_back(Class(2 * rem + fixed2, b.units));
            cls.push_back(Class(2 * b.self_tiles + fixed2, b.units));
            n_wg += (full + (rem > 0) + 1) * b.units;
        }
        if (n_wg > 64 * n_cu) continue;  // many rounds: any of the longer candidates is as good, and cheaper to price
        if (n_full > 0) cls.push_back(Class(2 * st + fixed2, n_full));
        std::sort(cls.begin(), cls.end(), std::greater<Class>());
        level.assign(1, Class(0, n_cu));  // a heap, the compute units that are free first on top
        int64_t t2 = 0;
        for (size_t c = 0; c < cls.size();) {
            int64_t left = 0;
            const int64_t cost = cls[c].first;
            while (c < cls.size() && cls[c].first == cost) left += cls[c++].second;
            while (left > 0) {
                Class now(level.front().first, 0);
                while (!level.empty() && level.front().first == now.first) {
                    now.second += level.front().second;
                    std::pop_heap(level.begin(), level.end(), std::greater<Class>());
                    level.pop_back();
                }
                const int64_t n = std::min(now.second, left);
                left -= n;
                level.push_back(Class(now.first + cost, n));
                std::push_heap(level.begin(), level.end(), std::greater<Class>());
                if (n < now.second) {
                    level.push_back(Class(now.first, now.second - n));
                    std::push_heap(level.begin(), level.end(), std::greater<Class>());
                }
                t2 = std::max(t2, now.first + cost);
            }
        }
        const double t = 0.5 * (double)t2 + per_wg * (double)n_wg;
        if (t < best_t) {
            best_t = t;
            best_st = st;
        }
    }
    return best_st;
}

}  // namespace adapshot
