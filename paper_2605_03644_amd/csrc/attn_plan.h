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
// Splits of a problem whose context is cut into pieces of split_tiles 64-key tiles.  The last one also takes the query's own
// tokens, unless these would give its wavefronts another step to run than the other splits have: then they are a
// split of their own.
inline int64_t stream_splits(const adapshot_model_desc& d, int64_t n_ctx, int64_t t_q, int64_t split_tiles) {
    const int64_t keys = split_tiles * 64, n = (n_ctx + keys - 1) / keys;
    if (n <= 1) return 1;
    if (n >= kStreamMaxSplits) return n;
    const int64_t sk = stream_step_keys(d), rest = n_ctx - (n - 1) * keys;
    const int64_t last = (rest + sk - 1) / sk + (t_q + sk - 1) / sk;
    return (last + kStreamWaves - 1) / kStreamWaves > (keys / sk + kStreamWaves - 1) / kStreamWaves ? n + 1 : n;
}

// What a launch of the streaming kernel takes, us, by its longest split (in 64-key tiles).  A workgroup spends 4.5 us before its
// first product and after its last one, and 0.6 us plus the loads of 82 KB/us for every round of its 8 wavefronts over its keys
// (bf16 x 128: 2.2 us per 256 keys; bf16 x 64 and fp32 x 64: 1.4 per 256 and 128; 1.1 over an assembled cache, 2 and more where the
// keys are gathered and rotated on the way, which is planned alike).  Splits cost their merge: 3 to 7 us where all workgroups fit
// the chip and share it, 9 where they do not and the last one to arrive does it (fp32 x 128, 64 tokens over 6k slots: 8 splits of
// 32 units 23.8 us, 10 splits 37.3).  So a problem gets the splits that fill the chip once, or none.  Measured / priced: 32/8 x 128,
// 24 tokens over 830 slots, 5 splits 9.8 / 11.5 (1: 12.3 / 13.3); 64 tokens over 1.7k, 2 splits 16.7 / 18.3 (1: 19.8 / 19.9); 1 token over
// 6.8k, 27 splits 10.4 / 11.2 (10: 13.5 / 14); 64 x bf16, 64 tokens over 2k, 4 splits 12.7 / 12.3 (1: 16.7 / 15.7); 4/2 x 64 fp32, 16 tokens over
// 250, 1 split 6.5 / 7.3 (4: 7.8 / 8.1), over 1000, 16 splits 7.9 / 8.7 (1: 13.6 / 15.7).
inline double stream_price(const adapshot_model_desc& d, int64_t n_cu, const StreamShape* shapes, int32_t n_shapes, int32_t row_blocks,
                           int64_t split_tiles) {
    const int64_t e = d.dtype == ADAPSHOT_BF16 ? 2 : 4, sk = stream_step_keys(d);
    const double round_us = 0.6 + (double)(kStreamWaves * sk * 2 * d.head_dim * e) / 82e3;
    int64_t units = 0, wgs = 0, read = 0, drawn = 0, longest = 0;  // tiles of a kv head: read by all workgroups, drawn from the memory
    for (int32_t i = 0; i < n_shapes; ++i) {
        const int64_t here = stream_units(d, shapes[i], row_blocks);
        units += here;
        wgs += here * std::max<int64_t>(1, (shapes[i].key_tiles + split_tiles - 1) / split_tiles);
        read += here * shapes[i].key_tiles;
        drawn += d.n_kv_heads * shapes[i].key_tiles;
        longest = std::max(longest, shapes[i].key_tiles);
    }
    const int64_t steps = std::min(split_tiles, longest) * 64 / sk, launch_rounds = (wgs + n_cu - 1) / n_cu;
    const double tile_mb = (double)(128 * d.head_dim * e) * 1e-6;
    const double t = (double)launch_rounds * (4.5 + (double)((steps + kStreamWaves - 1) / kStreamWaves) * round_us);
    // the memory gives more the more workgroups ask: 2.9 TB/s to 64 of them, 4.0 to 128, 5.1 to 256
    const double busy = (double)std::min(wgs, n_cu);
    const double loads = 4.5 + std::max((double)read * tile_mb / (0.045 * (double)n_cu), (double)drawn * tile_mb * (busy + 90.0) / (6.9 * busy));
    // (of plans that cost the same the one with more workgroups, up to the chip's)
    return std::max(t, loads) + (split_tiles >= longest ? 0.0 : launch_rounds == 1 ? 2.8 + 4.0 * (double)units / (double)n_cu : 9.0) -
           0.001 * busy;
}

// Split length (in 64-key tiles) of a launch: the longest context in n equal splits, the others in splits of the same length.
inline int64_t plan_stream_split_tiles(const adapshot_model_desc& d, int64_t n_cu, const StreamShape* shapes, int32_t n_shapes,
                                       int32_t row_blocks) {
    int64_t longest = 0;
    for (int32_t i = 0; i < n_shapes; ++i) longest = std::max(longest, shapes[i].key_tiles);
    if (longest == 0) return 1;
    const int64_t n_max = std::min<int64_t>(longest, kStreamMaxSplits);
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
// once per 256 rows and draws 6.1 TB/s, but is two launches (a batch: three), leaves wavefronts without rows idle and
// writes a partial for every split; the streaming kernel reads it once per 16 rows, in one launch.
// A batch goes to the streaming kernel if its items have at most 16 rows and its contexts at most twice kStreamBytes.  Per layer of
// a decode step (tile kernel with table copy and merge / streaming kernel, us): 28/4 heads, 6 queries of 16k slots 201 MB 50.0 / 44.6, 8
// 267 MB 62.1 / 57.4, 28 of 5k 282 MB 71.1 / 63.9, 12 of 16k 402 MB 84.7 / 84.2, 20 669 MB 130 / 132, 32 1067 MB 196 / 206; 32/8 heads, 16
// of 5k 323 MB 77.3 / 67.3.
constexpr int64_t kStreamBytes = 200000000;
inline bool stream_bytes_ok(const adapshot_model_desc& d, int64_t context_tokens) {
    return context_tokens * d.n_kv_heads * d.head_dim * 4 <= kStreamBytes;
}
// A single call compares prices.  The tile kernel's, fitted to calls of 64 to 512 rows over 250 to 5000 slots: 13 us for
// the two launches, 0.75 us per MB of partials, 0.65 or (more than 128 rows) 1 us per tile of a workgroup.  Us, tile /
// streaming: 32/8 heads, 8 tokens over 250 / 1.7k / 3.4k slots 14.0 / 14.5 / 15.6 and 10.7 / 10.4 / 11.2; 24 tokens over 830 / 3.4k
// 13.7 / 17.6 and 10.4 / 16.4; 64 tokens over 250 / 1.7k / 3.4k 14.6 / 23.5 / 24.6 and 10.1 / 17.6 / 24.5; 28/4 heads, 16 tokens over 5k
// 18.9 and 14.8, 64 tokens over 5k 24.5 and 32.1; 64/8 heads, 16 tokens over 5k 20.1 and 22.7.
inline bool single_by_tiles(const adapshot_model_desc& d, int32_t t_q, int64_t n_ctx, bool zero_copy, int64_t n_cu = 256) {
    if (!attn_mfma_supported(d)) return false;
    if (zero_copy || !stream_bytes_ok(d, n_ctx)) return true;  // (no gathered form of the streaming kernel for these models)
    const int64_t rows = (int64_t)t_q * (d.n_q_heads / d.n_kv_heads), key_tiles = (n_ctx + 63) / 64, self_tiles = ((int64_t)t_q + 63) / 64;
    // 1 token over 45k slots of 32/8 heads: 41.0 by tiles, 39.5 by streaming, shorter ones further apart; but from 100 MB on the
    // partials of more than 8 rows cost more than the second launch (4 tokens over 24k / 27k slots 27.9 / 30.5 and 26.5 / 35)
    if (rows <= 8) return false;
    if (rows > 16 * kAttnRowTile || !stream_bytes_ok(d, 2 * n_ctx)) return true;
    const StreamShape sh{rows, key_tiles + self_tiles};  // (the query's own tokens as more context)
    const int32_t rb = stream_row_blocks(d, n_cu, &sh, 1);
    const double stream = stream_price(d, n_cu, &sh, 1, rb, plan_stream_split_tiles(d, n_cu, &sh, 1, rb));
    const int64_t units = d.n_kv_heads * ((rows + kAttnRowTile - 1) / kAttnRowTile);
    const int64_t n_split = key_tiles > 0 ? plan_mfma_splits(n_cu, units, key_tiles, self_tiles) : 0;
    const int64_t per_wg = n_split > 0 ? (key_tiles + n_split - 1) / n_split : 0;
    const double drawn_mb = (double)(key_tiles * d.n_kv_heads * 256 * d.head_dim) * 1e-6;
    const double partials_mb = (double)((n_split + 1) * rows * d.n_kv_heads * d.head_dim * 2) * 1e-6;
    return 13.0 + 0.75 * partials_mb + std::max((rows > 128 ? 1.0 : 0.65) * (double)per_wg, drawn_mb / 6.1) < stream;
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
