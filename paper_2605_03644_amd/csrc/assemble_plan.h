// How the shots of an assembly reach its kernel.  Host logic over sizes alone -- no HIP types here, so that it can be compiled and checked
// without a GPU.
#pragma once
#include <stdint.h>

#include "adapshot.h"

namespace adapshot {

constexpr int kTileTok = 32;        // tokens of a tile, and slots of a workgroup, at most
constexpr int kAssembleBatch = 48;  // caches of a launch
// Launches that write more than the last-level cache holds: non-temporal stores, and lists of any length by blocks instead of tiles (below).
constexpr int64_t kAssembleStreamBytes = 256ll << 20;
// What kernel arguments hold: one cache and a list of kAssembleShots, or kAssembleFewCaches and kAssembleFewShots in all.
constexpr int kAssembleShots = 320;
constexpr int kAssembleFewCaches = 8, kAssembleFewShots = 272;
// A workgroup finds its shots in the arguments in three round trips more than a tile names them, which shows where it moves few bytes and the
// launch has many layers: rows of less than kAssembleNarrowRow bytes (workgroups of less than 16 KB).
constexpr int64_t kAssembleNarrowRow = 16384 / kTileTok;
constexpr int64_t kAssembleNarrowBlocks = 4096;
constexpr int32_t kAssembleNarrowLayers = 16;

// From this many layers on tiles are cut to the size of a workgroup (shot_tiles in adapshot_api.hip).
constexpr int kAssemblePieceLayers = 8;

enum AssembleRoute { kAssembleOneByArgs, kAssembleFewByArgs, kAssembleByList, kAssembleByTiles };

// One launch.  n_caches: those with tokens; n_runs: shots with tokens; n_blocks: workgroups of a layer and operand;
// n_tiles: tiles, or pieces of a workgroup's size.
//
// Lists that fit the kernel arguments go there: no pinned buffer, no event, no other kernel (2 caches of 16 shots 11.9 -> 11.2 us, 4 of
// 64 short ones 19.4 -> 14.8).  Not batches of narrow rows in launches of many workgroups or layers (us, tiles / arguments, 2 x 64
// bf16 heads: 8 layers, 27 MB written 15.6 / 14.2, 110 MB 46.7 / 46.0, 772 MB 295 / 307; 28 layers, 17 MB 11.1 / 11.9, 234 MB 84.7 / 89.0; 1 x 64: 8
// layers, 14 MB 11.8 / 10.5, 33 MB 19.9 / 21.7, 28 layers, 48 MB 26.2 / 29.8; 2 x 16: 4 layers 15 MB 20.5 / 14.4, 28 layers 97 MB 70 / 88).
//
// A longer one goes through device memory where the launch writes more than the last-level cache holds, else as tiles: the kernel ahead of
// the launch costs 4 to 7 us, and what it saves grows with the bytes.  MB written, by tiles / by list, us: one layer 171 57.6 / 61.6, 217 71.9
// / 74.9, 341 130.2 / 129.0, 549 207 / 200, 1759 732 / 630; two layers 108 42.0 / 44.2, 269 104.7 / 105.2, 407 156 / 153, 1066 396 / 376;
// 8 layers 2113 770 / 751, 28 layers 7441 2708 / 2618.  (Lists cut into launches with arguments: each costs 4.5 us.)  Up to twice that it saves
// nothing where tiles leave little undone: fp32 models with shots of more than a tile (8 x 128, one layer, shots of 104 tokens, 283 MB 106.5 / 109.3;
// of 25, 304 MB 130.8 / 116.8), and 8 layers and more, whose tiles are whole workgroups, unless these are mostly empty (2 x 64 fp32, 8 layers,
// shots of 25 tokens, 304 MB 108.3 / 113.6; 4 x 128 bf16, 28 layers, 2.5 tokens, 287 MB 138 / 112) or rows are a few bytes (1 x 16, 28 layers, 276
// MB 361 / 275).
inline AssembleRoute assemble_route(const adapshot_model_desc& d, int64_t n_caches, int64_t n_runs, int64_t n_tok, int64_t n_blocks,
                                    int64_t n_tiles) {
    const int64_t row_bytes = (int64_t)d.n_kv_heads * d.head_dim * (d.dtype == ADAPSHOT_F32 ? 4 : 2);
    if (n_caches == 1 && n_runs <= kAssembleShots) return kAssembleOneByArgs;
    if (n_caches <= kAssembleFewCaches && n_runs <= kAssembleFewShots &&
        (row_bytes >= kAssembleNarrowRow || (d.n_layers < kAssembleNarrowLayers && n_blocks * d.n_layers <= kAssembleNarrowBlocks)))
        return kAssembleFewByArgs;
    const int64_t written = 2 * n_tok * row_bytes * d.n_layers;
    const bool soon = row_bytes < kAssembleNarrowRow / 2 ||
                      (d.n_layers >= kAssemblePieceLayers ? n_tiles >= 4 * n_blocks : d.dtype == ADAPSHOT_BF16 || 2 * n_tok < 3 * kTileTok * n_runs);
    return written > (soon ? 1 : 2) * kAssembleStreamBytes ? kAssembleByList : kAssembleByTiles;
}

}  // namespace adapshot
