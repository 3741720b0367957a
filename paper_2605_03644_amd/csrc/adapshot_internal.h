// Internal declarations shared by the host API and the kernel translation units.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "adapshot.h"
#include "assemble_plan.h"
#include "attn_plan.h"

namespace adapshot {

// ---- RoPE tables --------------------------------------------------------------
// Angle multiplier a (a position or a position offset) is split as a = 64*hi + lo.
// tab_hi[hi][i] = (cos, sin)(64*hi*theta_i), tab_lo[lo][i] = (cos, sin)(lo*theta_i),
// both evaluated in fp64 and rounded once to fp32.  cos/sin(a*theta_i) follows by one
// angle addition in fp32 (error ~3e-7 absolute), see Eq. (rope_compensation).  The rows of tab_lo from kRopeLo on are those
// of lo + 1/2, which the zero-copy attention uses: a tile of 64 keys lies symmetrically around its centre.
constexpr int kRopeLoBits = 6;
constexpr int kRopeLo = 1 << kRopeLoBits;

// Division of n in [0, 2^31) by a fixed d >= 1: with s = ceil(log2 d), n / d = n * ceil(2^(31 + s) / d) >> (31 + s), exactly, as the
// rounded-up factor is off by less than 2^-31 of itself per unit of n.  (A division by a kernel argument is 30 dependent instructions.)
struct FastDiv {
    uint32_t mul;
    int32_t shift;
    __device__ __forceinline__ int of(int n) const { return (int)(__umulhi((unsigned)n << 1, mul) >> shift); }
};
inline FastDiv fast_div(int32_t d) {
    int32_t s = 0;
    while (((int64_t)1 << s) < d) ++s;
    return FastDiv{(uint32_t)((((uint64_t)1 << (31 + s)) + (uint64_t)d - 1) / (uint64_t)d), s};
}

// ---- assemble -------------------------------------------------------------------
// One tile = up to kTileTok consecutive tokens of ONE shot: contiguous in the pool
// and contiguous in the cache.  Angle of token tau in the tile: angle0 + tau*angle_step.
// A launch serves up to kAssembleBatch caches: a tile names its cache, and the caches'
// buffers travel in the kernel arguments.
struct TileDesc {
    int32_t src_tok;     // first pool token (index inside a layer)
    int32_t dst_slot;    // first cache slot; the token's new position is the cache's pos0 + slot
    int32_t angle0;      // angle multiplier of the first token
    int32_t n_tok;       // 1..kTileTok
    int32_t angle_step;  // 1: keys un-rotated (angle = position); 0: rotated at local positions (angle = shot offset)
    int32_t shot;        // pool shot id
    int32_t tok0;        // index of the first token inside its shot
    int32_t cache;       // index into AssembleParams::dst
};
static_assert(sizeof(TileDesc) == 32, "TileDesc is read as two 16-byte words");

struct AssembleDst {  // one cache of the launch
    char* k_out;
    char* v_out;
    int32_t* slot_shot;
    int32_t* slot_tok;
    int64_t* slot_pos;
    int64_t layer_stride_bytes;
    int64_t pos0;
};

struct AssembleParams {
    const char* k_pool;
    const char* v_pool;
    const TileDesc* tiles;  // pinned host memory, read by the kernel
    const float2* tab_lo;
    const float2* tab_hi;
    int64_t pool_layer_stride_bytes;
    int64_t n_tokens;      // tokens of all tiles together
    int32_t n_tiles;
    int32_t n_layers;
    int32_t n_dst;         // caches of this launch (entries of dst in use)
    int32_t wg_tok;        // tokens of a tile per workgroup: a power of two <= kTileTok (kTileTok / wg_tok workgroups per tile;
                           // kTileTok: the host has cut the shots into one-workgroup tiles already)
    int32_t n_kv_heads;
    int32_t head_dim;
    int32_t dtype;
    AssembleDst dst[kAssembleBatch];
};
hipError_t launch_assemble(const AssembleParams& p, hipStream_t stream);

// Without tiles: workgroups are cut by cache slots, wg_tok consecutive ones each, cache after cache, and look their shots up.
struct ShotRun {
    int32_t slot;     // first slot of the shot, counted from the call's first slot in this cache; increasing, the first one 0
    int32_t src_tok;  // its first pool token (index inside a layer)
    int32_t shot;     // pool shot id
};
struct ShotsDst : AssembleDst {
    int32_t slot0;         // first slot of the call
    int32_t n_tokens;      // > 0
    int32_t run0, n_runs;  // its part of the list
    int32_t block0;        // its first workgroup of the launch, of every layer
    int32_t pad;
};
// A launch whose list does not fit the kernel arguments finds both in device memory, written by a kernel ahead of it: the runs, and for
// every workgroup what it would look up.
struct AssembleBlock {
    int32_t src_tok;  // pool token of its first slot
    int32_t run;      // the run of that slot
    int32_t skip;     // slots of the run before it
    int32_t what;     // cache | kBlockOneRun: all its slots are the run's
};
constexpr int32_t kBlockOneRun = 1 << 8;
struct ListRun {
    ShotRun run;
    int32_t cache;
};
struct ShotsHead {
    const char* k_pool;
    const char* v_pool;
    const float2* tab_lo;
    const float2* tab_hi;
    int64_t pool_layer_stride_bytes;
    const ListRun* host_list;  // pinned host memory, read by the kernel that writes the next two
    ListRun* list;             // device memory
    AssembleBlock* blocks;
    int64_t n_tokens;     // of all caches together
    int32_t n_caches, n_layers, n_blocks, n_runs;
    int32_t wg_tok;  // slots of a workgroup: a power of two <= kTileTok
    int32_t local;   // 1: keys rotated at local positions (angle = position of the shot's first slot), 0: un-rotated (angle = position)
    int32_t n_kv_heads, head_dim, dtype;
};
// Kernel arguments end at 4 KB: one cache and a list of kAssembleShots, kAssembleFewCaches and kAssembleFewShots in all, or
// kAssembleBatch caches and the list in device memory (NS = 0).
static_assert(kAssembleBatch <= kBlockOneRun, "a block's cache");
template <int NC, int NS>
struct AssembleShotsParams {
    ShotsHead h;
    ShotsDst dst[NC];
    ShotRun shots[NS > 0 ? NS : 1];
};
typedef AssembleShotsParams<1, kAssembleShots> AssembleOne;
typedef AssembleShotsParams<kAssembleFewCaches, kAssembleFewShots> AssembleFew;
typedef AssembleShotsParams<kAssembleBatch, 0> AssembleMany;
static_assert(sizeof(AssembleOne) <= 4096 && sizeof(AssembleFew) <= 4096 && sizeof(AssembleMany) <= 4096, "kernel arguments");
hipError_t launch_assemble_shots(const AssembleOne& p, hipStream_t stream);
hipError_t launch_assemble_shots(const AssembleFew& p, hipStream_t stream);
hipError_t launch_assemble_shots(const AssembleMany& p, hipStream_t stream);
hipError_t launch_assemble_list(const AssembleMany& p, hipStream_t stream);  // ahead of the last one: list and blocks from host_list

// One decode step: cache i of this launch receives token row [layer][first + i] of k_new / v_new at
// slot[i], the key rotated to pos[i].  Pointer tables travel in the kernel arguments.
constexpr int kDecodeBatch = 32;
struct DecodeAppendParams {
    const char* k_new;  // [n_layers][n_total][h_kv][d], un-rotated
    const char* v_new;
    const float2* tab_lo;
    const float2* tab_hi;
    char* k_out[kDecodeBatch];
    char* v_out[kDecodeBatch];
    int32_t* slot_shot[kDecodeBatch];
    int32_t* slot_tok[kDecodeBatch];
    int64_t* slot_pos[kDecodeBatch];
    int32_t capacity[kDecodeBatch];
    int32_t slot[kDecodeBatch];
    int32_t pos[kDecodeBatch];
    int32_t n_layers, n_kv_heads, head_dim, dtype;
    int32_t n_total, first, count;
};
hipError_t launch_decode_append(const DecodeAppendParams& p, hipStream_t stream);

// ---- attention --------------------------------------------------------------------
struct RopeRowsParams {
    const void* q;       // [t_q][h_q][d]
    void* q_rot;         // [t_q][h_q][d], scaled by log2(e)/sqrt(d)
    const float2* tab_lo;
    const float2* tab_hi;
    int64_t q_pos0;
    int32_t t_q, n_q_heads, head_dim, dtype;
    float q_scale;
};
hipError_t launch_rope_rows(const RopeRowsParams& p, hipStream_t stream);

// Split plan: splits 0..n_split-1 cover context keys [s*keys_per_split, ...) and
// split n_split is the causal self part.  Partials are indexed [split][kv head][row]
// with row = j*g + (h % g).
// What only the MFMA kernel's prologue (and its zero-copy form) reads.  Kept apart from AttnParams so that none
// of it occupies scalar registers during the key loop.
struct AttnFold {
    // The kernel rotates the rows it needs itself (Eq. rope_encoding at position q_pos0 + j), the query rows
    // scaled by q_scale = log2(e)/sqrt(d) on the way into its fragments, the query's own keys on the way into LDS.
    const void* q_raw;       // [t_q][h_q][d] as the caller gave it
    const void* k_self_raw;  // [t_q][h_kv][d] as the caller gave it
    const float2* tab_lo;
    const float2* tab_hi;
    int64_t q_pos0;
    float q_scale;
    int32_t pool_tokens;  // zero-copy form: tokens in a pool layer (gathered rows are clamped to it)
    // Zero-copy form (template parameter POOL): k_cache / v_cache are the POOL's layer, context slot u holds pool
    // token slot_src[u], and its key is rotated to position pos0 + u inside the key loop;
    // row i of tile_rot, 64 entries, holds (cos, sin)((pos0 + 64 i + 31.5) theta_f), the centre of 64-slot tile i, in the order
    // of tile_rot_place().  slot_src is 16-byte
    // aligned and readable for 256 entries past the context's last slot (the kernel fetches it 1 KB at a time).
    const int32_t* slot_src;
    const float2* tile_rot;
};

struct AttnParams {
    const void* k_cache;  // one layer [>=n_ctx][h_kv][d]
    const void* v_cache;
    const void* v_self;
    // Partials, indexed [n_split+1][h_kv][rows]: part_mlf = (reference maximum in log2 units, row sum l, factor f = l * a,
    // unused) and a row O' of d fp16 values with  sum_k p_k v_k = f * O':  O' = accumulator / (l * a), a = the largest
    // |accumulator| / l of the row, so |O'| <= 1 whatever the range of V; error per element <= 2^-11 of the row's largest
    // partial output.
    void* part_o;
    float4* part_mlf;
    void* out;       // [t_q][h_q][d]
    int64_t n_ctx;
    int64_t keys_per_split;
    int32_t n_split;
    int32_t t_q, n_q_heads, n_kv_heads, head_dim, dtype;
    // Batched launches only: k_cache / v_cache point at layer 0 of the item's context and the launch names the
    // layer, so that the tables of a batch serve every layer of a model (0 for single calls).
    int64_t layer_stride_bytes;
};
// ---- streaming attention (attn_stream_kernel.h): every shape the 256-row tile kernel does not cover -------------
struct StreamItem {
    const char* q;
    const char* k_self;
    const char* v_self;
    char* out;
    const char* k_ctx;  // one layer of the context (assembled cache or pool)
    const char* v_ctx;
    int32_t n_ctx, t_q, q_pos0;
    int32_t keys_per_split, n_split;  // the last split also takes the query's own tokens
    int32_t unit0;      // first unit of the problem in the workspaces
    int32_t block0;     // its first workgroup in the launch
    FastDiv div_split;  // by n_split
};
template <int NI>
struct StreamArgs {
    const float2* tab_lo;
    const float2* tab_hi;
    float* part_o;       // [unit][max_split][16 NR rows][d] fp32, unnormalised (launches with splits)
    float* part_ml;      // [unit][max_split][16 NR rows] (m, l)
    unsigned* counters;  // [unit * counter_stride], zero between launches
    const int32_t* slot_src;  // zero-copy form: context slot -> pool token (null: the context is an assembled cache)
    int64_t ctx_pos0;         // zero-copy form: position of context slot 0
    int32_t n_q_heads, n_kv_heads, g, max_split, pool_tokens, counter_stride;
    FastDiv div_hkv, div_g;
    float q_scale;
    StreamItem it[NI];
};
struct StreamLaunch {
    const float2* tab_lo;
    const float2* tab_hi;
    float* part_o;
    float* part_ml;
    unsigned* counters;
    const int32_t* slot_src;
    int64_t ctx_pos0;
    int32_t n_q_heads, n_kv_heads, head_dim, dtype, max_split, pool_tokens, counter_stride;
    int32_t row_blocks;  // 16-row blocks per workgroup: 1 or 2
    int32_t n_wgs;       // workgroups of all problems
    int32_t n_items;
    float q_scale;
    const StreamItem* items;
};
hipError_t launch_attn_stream(const StreamLaunch& s, hipStream_t stream);
hipError_t launch_attn_stream_f32(const StreamLaunch& s, hipStream_t stream);
hipError_t launch_attn_stream_bf16(const StreamLaunch& s, hipStream_t stream);
hipError_t launch_attn_mfma(const AttnParams& p, const AttnFold& f, hipStream_t stream);
hipError_t launch_attn_mfma_pool(const AttnParams& p, const AttnFold& f, hipStream_t stream);  // zero-copy form
// Place of frequency f in a row of tile_rot: those of a lane's four, 4 c .. 4 c + 3, are 16 bytes of either half of the row.
__device__ __forceinline__ int tile_rot_place(int f) { return ((f >> 1) & 1) * 32 + (f >> 2) * 2 + (f & 1); }
// Expands the per-shot segments of a zero-copy context into slot_src and builds tile_rot (head_dim 128).
struct PoolSeg {
    int32_t slot0, src_tok0, len, pad;
};
struct PoolPlanParams {
    const PoolSeg* segs;  // pinned host memory, read by the kernel
    int32_t* slot_src;
    float2* tile_rot;
    const float2* tab_lo;
    const float2* tab_mid;
    int64_t pos0;
    int32_t n_segs, n_tiles, head_dim;
};
hipError_t launch_pool_plan(const PoolPlanParams& p, hipStream_t stream);
hipError_t launch_attn_combine(const AttnParams& p, hipStream_t stream);

// ---- a batch of attention problems in two launches (attend, combine) ------------------------
// The tables live in device memory for the duration of the launches; every workgroup reads its own
// entry.  The probes of one query over nested prefixes of one cache, the queries of a decode step and
// the queries of a probe sweep are all such batches (Probe-based Dynamic Evaluation).
struct AttnBatchItem {
    AttnParams attn;
    AttnFold fold;
};
struct AttnWork {  // one workgroup of the batched MFMA kernel
    int32_t item, hk, row_tile, split;
};
struct CombineWork {  // one workgroup of the batched combine kernel: 16 (kv head, row) pairs from pair0 on (fp16 partials)
    int32_t item, pair0;
};
// A smaller batch travels in the kernel arguments, which costs neither the table copy (4.2 us) nor the wait of the kernel behind it for its
// completion event (4.5 us): a decode step of 32 queries of 16k slots 185 -> 180 us a layer, passes of probe sweeps over one to
// three layers 235 -> 203 and 170 -> 145.  What goes beyond them is as before: 24 tokens of 32/8 heads over 1k slots, 32 items 51.6 ->
// 46.5 us, 33 items 67.  An entry of work is an (item, split, row tile), served by n_kv_heads workgroups, the
// kv head fastest as in the tables.  Kernel arguments end at 4 KB.
constexpr int kBatchArgItems = 32, kBatchArgWork = 352;
struct BatchArgItem {
    const void* q;
    const void* k_self;
    const void* v_self;
    const void* k_ctx;  // one layer of the context; zero-copy form: of the pool
    const void* v_ctx;
    const int32_t* slot_src;  // zero-copy form
    int32_t n_ctx, q_pos0, t_q, keys_per_split, n_split;
    int32_t part_row0;  // first row of the item's partials
};
struct BatchArgs {
    void* part_o;      // rows of fp16 values, [item][n_split + 1][h_kv][rows]
    float4* part_mlf;
    const float2* tab_lo;
    const float2* tab_hi;
    const float2* tile_rot;
    int32_t n_q_heads, n_kv_heads, pool_tokens;
    float q_scale;
    FastDiv div_hkv;
    BatchArgItem it[kBatchArgItems];
    uint32_t work[kBatchArgWork];
};
inline uint32_t batch_work(int32_t item, int32_t split, int32_t row_tile) { return (uint32_t)(item | split << 5 | row_tile << 12); }
constexpr int32_t kBatchArgRowTiles = 1 << 20;
static_assert(kBatchArgItems <= 32 && sizeof(BatchArgs) <= 4096, "work entries, kernel arguments");
struct CombineArgs {
    const void* part_o;
    const float4* part_mlf;
    int32_t n_q_heads, n_kv_heads;
    struct {
        void* out;
        int32_t part_row0, t_q, n_split;
        int32_t block0;  // the item's first workgroup
    } it[kBatchArgItems];
};
hipError_t launch_attn_mfma_batch_args(const BatchArgs& a, int n_wgs, bool pool, bool stream_tiles, hipStream_t stream);
hipError_t launch_attn_combine_batch_args(const CombineArgs& a, int n_wgs, int max_partials, hipStream_t stream);
// Tables written by the host into pinned memory are brought to device memory by a kernel (a DMA copy
// between two kernels of a stream costs more than the copy itself).  bytes is a multiple of 16.
hipError_t launch_copy_table(void* dst, const void* src_pinned, size_t bytes, hipStream_t stream);
// stream_tiles: no two items read the same context and none has more than kAttnStreamRows rows per kv head
hipError_t launch_attn_mfma_batched(const AttnBatchItem* items, const AttnWork* work, int n_work, bool pool,
                                    bool stream_tiles, int layer, hipStream_t stream);
// max_partials: the most partial rows that any item merges per output row (its context splits + 1)
hipError_t launch_attn_combine_batched(const AttnBatchItem* items, const CombineWork* work, int n_work, int max_partials,
                                       hipStream_t stream);

// ---- relevance ranking over the pool (Eq. attention_score) ----------------------------------
// The query rows meet the locally encoded keys of ALL pool tokens at one layer.  The pool is cut into equal splits of
// consecutive keys; a SEGMENT is what one split holds of one shot (a shot that a split boundary cuts has two), and the
// key pass leaves the exponentials of every (segment, row) summed, relative to the row's reference maximum in its split.
struct RankPrepareParams {
    const char* k_pool;       // one layer [tokens][h_kv][d], un-rotated
    char* k_out;              // same layout, every key rotated to its position inside its shot
    const int32_t* shot_off;  // [n_shots + 1] first token of every shot
    const float2* tab_lo;
    const float2* tab_hi;
    int64_t max_len;          // longest shot
    int32_t n_shots, n_kv_heads, head_dim;
};
hipError_t launch_rank_prepare(const RankPrepareParams& p, hipStream_t stream);
struct RankScoreParams {
    const void* k;            // one layer [tokens][h_kv][128], keys as a cache holds them
    const void* q;            // [t_q][h_q][128] as the caller gave it; rotated to q_pos0 + j here
    const float2* tab_lo;
    const float2* tab_hi;
    const int32_t* seg_end;     // [n_seg] one past the segment's last key
    const int32_t* split_seg0;  // [n_split + 1] first segment of every split
    const uint32_t* end_bits;   // a bit per key from key0 on: a segment ends with it
    float* part;              // [n_seg][pairs], pair = kv head * rows + row
    float2* part_ml;          // [n_split][pairs] (reference maximum in log2 units, row sum)
    int64_t q_pos0;
    float q_scale;
    int32_t key0, n_tok;      // keys [key0, n_tok)
    int32_t keys_per_split;   // multiple of 64
    int32_t n_split, t_q, n_q_heads, n_kv_heads;
    int32_t n_seg;
};
hipError_t launch_rank_scores(const RankScoreParams& p, hipStream_t stream);
struct RankReduceParams {
    const float* part;        // [n_seg][pairs]
    const float2* part_ml;    // [n_split][pairs]
    float* weights;           // [n_split][pairs] scratch
    float* scores;            // [n_shots]
    const int32_t* seg_split;  // [n_seg] split of every segment
    const int32_t* shot_seg0;  // [n_shots + 1] first segment of every shot
    const float* inv_len;     // [n_shots] 1 / T_i
    float inv_rows;           // 1 / (t_q * n_q_heads)
    int64_t n_pairs;
    int32_t n_split, n_shots;
};
hipError_t launch_rank_weights(const RankReduceParams& p, hipStream_t stream);  // merge weights of the splits
hipError_t launch_rank_reduce(const RankReduceParams& p, hipStream_t stream);   // weighted sums, one shot per workgroup

// Ranking for the shapes the matrix-core kernel does not cover: one wavefront per (query token, head) walks the
// whole pool layer twice (normaliser, then the mass of every shot), a second kernel adds the rows in a fixed order.
struct RankGenericParams {
    const void* k_pool;       // one layer [tokens][h_kv][d]
    const void* q_rot;        // [t_q][h_q][d] rotated to q_pos0 + j, scaled by log2(e)/sqrt(d)
    const int64_t* shot_off;  // DEVICE [n_shots + 1]
    const float2* tab_lo;
    const float2* tab_hi;
    float* mass;              // [t_q * h_q][n_shots] scratch: attention received by every shot from one row
    float* scores;            // [n_shots]
    int32_t n_shots, t_q, n_q_heads, n_kv_heads, head_dim, dtype, key_state;
};
hipError_t launch_rank_generic(const RankGenericParams& p, hipStream_t stream);

// ---- entropy ------------------------------------------------------------------------
struct EntropyParams {
    const float* logits;
    float* out;
    float* partials;  // [n_rows][n_chunks][3] = (max, sum exp, sum (z-max) exp)
    unsigned* counters;  // [n_rows * counter_stride], zero between launches (the one-launch form)
    int64_t row_stride;
    int32_t n_rows, vocab, chunk, n_chunks, counter_stride;
};
// The file-scope device array behind adapshot_probe_entropy_static: room for this many (row, chunk) partials.
constexpr int kStaticEntropyPartials = 65536;
// Device address of that array on the CURRENT device (looked up once per device, then remembered).
hipError_t entropy_static_scratch(float** out);
inline bool entropy_rows_aligned(const float* logits, int64_t row_stride) {  // for 16-byte loads
    return ((uintptr_t)logits & 15u) == 0 && row_stride % 4 == 0;
}
hipError_t launch_entropy_chunk(const EntropyParams& p, hipStream_t stream);
// Eq. (entropy) over a set C of answer tokens, from the same vocabulary-wide partials.
constexpr int kMaxAnswerTokens = 16;
struct AnswerTokens {
    int32_t n;
    int32_t mode;  // ADAPSHOT_ENTROPY_FULL_P / ADAPSHOT_ENTROPY_RENORMALISED
    int32_t id[kMaxAnswerTokens];
};
hipError_t launch_entropy_finish(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream);
// Up to this many rows of several chunks merge in the launch that reduces the chunks.  More rows have counters closer than
// a line and arrivals that cost what a second launch does (one launch / two, us: 600 x 16000 12.1 / 12.7, 1000 x 10000 13.8 /
// 14.4, 2000 x 10000 22.0 / 21.4, 4096 x 16383 49.4 / 47.8; a workgroup per row / two launches: 5000 x 16001 74.4 / 67.4,
// 20000 x 9000 177 / 147).
constexpr int32_t kEntropyFusedRows = 1024;
// Chunks and their merge in one launch; c == nullptr: the vocabulary-wide entropy.
hipError_t launch_entropy_fused(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream);
// Whole rows in one launch (one workgroup per row); c == nullptr: the vocabulary-wide entropy.
hipError_t launch_entropy_rows(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream);

// ---- host-side helpers -----------------------------------------------------------------
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    hipError_t reserve(size_t need, std::vector<void*>& retired);  // grow-only; an outgrown buffer is parked in `retired`
    void release();
};

struct PinnedRing {
    static constexpr int kSlots = 8;
    void* host[kSlots] = {};
    size_t bytes[kSlots] = {};
    hipEvent_t ev[kSlots] = {};
    bool pending[kSlots] = {};
    int next = 0;
    // Returns a pinned buffer of at least `need` bytes that no enqueued kernel still reads.
    hipError_t acquire(size_t need, int* slot, void** ptr);
    // `launch` enqueues one kernel that reads the slot: nobody writes the slot before it has finished.
    template <typename F>
    hipError_t launch_reader(int slot, hipStream_t stream, F&& launch);
    void release();
};

// Timing events of the launch in progress.  When set, launch_kernel attaches them to the dispatch itself
// (hipExtLaunchKernelGGL): their difference is then the kernel's own execution time as its completion
// signal records it, without the two command-processor round trips that events recorded around a launch
// add (about 2.5 us on this part).  One dispatch consumes the pair, or a stop event that comes alone.
struct LaunchEvents {
    hipEvent_t start = nullptr, stop = nullptr;
};
extern thread_local LaunchEvents g_launch_events;

template <typename... KArgs, typename... Args>
inline void launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, hipStream_t stream, Args&&... args) {
    static_assert(sizeof...(KArgs) == sizeof...(Args), "one argument per kernel parameter");
    if (g_launch_events.stop) {
        const LaunchEvents ev = g_launch_events;
        g_launch_events = LaunchEvents{};
        hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, ev.start, ev.stop, 0, static_cast<KArgs>(args)...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, 0, stream, static_cast<KArgs>(args)...);
    }
}

// The event is the dispatch's own completion where that is possible: recorded behind the kernel it is a packet of its own, which
// the next kernel waits for.  Recorded / attached, us: sweeps of 7 queries over one layer 152.2 / 146.0, of one query over two
// layers 129.3 / 121.5; 32 decode queries of 16k slots the same (a table copy in 185 us).  Not in a capture, where it stays a node, nor in a
// launch that carries timing events already.
template <typename F>
hipError_t PinnedRing::launch_reader(int slot, hipStream_t stream, F&& launch) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    const bool known = hipStreamIsCapturing(stream, &capture) == hipSuccess;
    if (!known) (void)hipGetLastError();
    const bool attach = !g_launch_events.stop && known && capture == hipStreamCaptureStatusNone;
    if (attach) g_launch_events.stop = ev[slot];
    hipError_t e = launch();
    const bool attached = attach && !g_launch_events.stop;
    if (attach) g_launch_events.stop = nullptr;
    if (e == hipSuccess && !attached) e = hipEventRecord(ev[slot], stream);
    if (e == hipSuccess) pending[slot] = true;
    return e;
}

// Optional per-kernel timing with HIP events on the launch stream (measurement aid).
struct Profiler {
    struct Rec {
        int kind;
        hipEvent_t start, stop;
    };
    bool on = false;
    std::vector<Rec> recs;
    std::vector<hipEvent_t> free_events;
    hipError_t begin(int kind, hipStream_t stream);
    hipError_t end(hipStream_t stream);
    void release();
};

}  // namespace adapshot

struct adapshot_ctx {
    adapshot_model_desc desc;
    int device = -1;
    int elem_bytes = 0;
    int64_t row_bytes = 0;  // n_kv_heads * head_dim * elem_bytes
    int64_t max_position = 0;
    // pool
    const void* k_pool = nullptr;
    const void* v_pool = nullptr;
    std::vector<int64_t> shot_offsets;
    int64_t pool_layer_stride_tokens = 0;
    int32_t n_shots = 0;
    // tables
    float2* tab_lo = nullptr;
    float2* tab_hi = nullptr;
    float2* tab_mid = nullptr;  // (cos, sin)((64 i + 31.5) theta_f), where the tile kernel serves the model
    unsigned* stream_counters = nullptr;  // arrival counters of split streaming launches, zero between launches
    float* static_ent = nullptr;  // this device's copy of the static entropy scratch array (not owned)
    // scratch
    adapshot::PinnedRing tile_ring;
    adapshot::DevBuf run_lists;  // shot lists of assemble calls, run_list_bytes for every slot of tile_ring
    size_t run_list_bytes = 0;
    adapshot::DevBuf q_rot, part_o, part_ml, ent_part, batch_tab, pool_src, pool_rot;
    // What the device-side tables of the last batched attention call (batch_tab) and of the last zero-copy plan
    // (pool_src, pool_rot) were built from: a call with the same inputs -- the next layer of the same batch --
    // reuses them instead of planning and uploading again.  Empty = nothing to reuse.
    std::vector<unsigned char> batch_key, pool_key;
    // (a batch in the kernel arguments keeps those: the contexts' layer 0 and strides are beside them)
    bool batch_by_args = false;
    adapshot::BatchArgs batch_args;
    adapshot::CombineArgs batch_comb;
    struct {
        const char *k0, *v0;
        int64_t layer_stride_bytes;
    } batch_ctx[adapshot::kBatchArgItems];
    int64_t batch_n_attn = 0, batch_n_comb = 0;
    int32_t batch_max_partials = 0;
    size_t batch_attn_off = 0, batch_comb_off = 0;
    // ranking state of one pool layer, built on first use
    int32_t rank_layer = -1;
    int32_t rank_n_split = 0, rank_n_seg = 0, rank_keys_per_split = 0;
    adapshot::DevBuf rank_k, rank_tab, rank_w;
    const int32_t* rank_seg_end = nullptr;    // views into rank_tab
    const int32_t* rank_seg_split = nullptr;
    const int32_t* rank_split_seg0 = nullptr;
    const int32_t* rank_shot_seg0 = nullptr;
    const uint32_t* rank_end_bits = nullptr;
    const float* rank_inv_len = nullptr;
    std::vector<void*> retired;  // outgrown workspaces, freed when the context is destroyed
    adapshot::Profiler prof;
    int n_cu = 256;
    int32_t assemble_wg_tok = adapshot::kTileTok;  // tokens of a tile per assemble workgroup
    int32_t force_splits = 0;  // adapshot_set_attn_splits: 0 = the planner chooses
    int32_t entropy_rows_min = 256;  // from this many rows on, probe entropy runs one workgroup per row in one launch
    std::string last_error;
};
