// Query-over-cache attention, what surrounds the tile kernel:
//   rope_rows     -- rotate the query rows to positions q_pos0 + j (Eq. rope_encoding)
//                    and fold the softmax scale log2(e)/sqrt(d) (Eq. attention_score's
//                    1/sqrt(d)) into them, for ranking (the attention kernels rotate
//                    their rows themselves);
//   attn_combine  -- merges the per-split (max, sum, scaled output) partials of the
//                    tile kernel.
#include <algorithm>

#include "adapshot_internal.h"

namespace adapshot {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned short f32_to_bf16_rne(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(unsigned short, b);
}

// ---- rope_rows ----------------------------------------------------------------------
// One thread per pair of 16-byte chunks holding rotation partners (i, i + d/2), i = NP*ci .. NP*ci + NP - 1.
template <int DTYPE>
__device__ __forceinline__ void rope_rows_block(const RopeRowsParams& p, int64_t block) {
    constexpr int NP = DTYPE == ADAPSHOT_BF16 ? 8 : 4;  // pairs per chunk
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const int half = p.head_dim >> 1;
    const int cpr = half / NP;  // chunk pairs per row
    const int64_t idx = block * 256 + threadIdx.x;
    if (idx >= (int64_t)p.t_q * p.n_q_heads * cpr) return;
    const int64_t r = idx / cpr;
    const int ci = (int)(idx - r * cpr);
    const int j = (int)(r / p.n_q_heads);
    const int64_t a = p.q_pos0 + j;
    const float2* th = p.tab_hi + (a >> kRopeLoBits) * half + ci * NP;
    const float2* tl = p.tab_lo + (a & (kRopeLo - 1)) * half + ci * NP;
    const char* src = (const char*)p.q;
    char* dst = (char*)p.q_rot;
    const int64_t o = (r * p.head_dim + ci * NP) * (DTYPE == ADAPSHOT_BF16 ? 2 : 4);
    const int64_t ho = (int64_t)half * (DTYPE == ADAPSHOT_BF16 ? 2 : 4);
    u32x4 x1 = *(const u32x4*)(src + o), x2 = *(const u32x4*)(src + o + ho);
    const float sc = p.q_scale;
    float y1[NP], y2[NP];
#pragma unroll
    for (int w = 0; w < NP; ++w) {
        const float2 h = th[w], l = tl[w];
        const float c = h.x * l.x - h.y * l.y;
        const float s = h.y * l.x + h.x * l.y;
        float a1, a2;
        if (DTYPE == ADAPSHOT_BF16) {
            const unsigned w1 = x1[w >> 1], w2 = x2[w >> 1];
            a1 = (w & 1) ? __uint_as_float(w1 & 0xffff0000u) : __uint_as_float(w1 << 16);
            a2 = (w & 1) ? __uint_as_float(w2 & 0xffff0000u) : __uint_as_float(w2 << 16);
        } else {
            a1 = __uint_as_float(x1[w]);
            a2 = __uint_as_float(x2[w]);
        }
        y1[w] = (a1 * c - a2 * s) * sc;
        y2[w] = (a2 * c + a1 * s) * sc;
    }
    if (DTYPE == ADAPSHOT_BF16) {
#pragma unroll
        for (int w = 0; w < NP; w += 2) {
            x1[w >> 1] = (unsigned)f32_to_bf16_rne(y1[w]) | ((unsigned)f32_to_bf16_rne(y1[w + 1]) << 16);
            x2[w >> 1] = (unsigned)f32_to_bf16_rne(y2[w]) | ((unsigned)f32_to_bf16_rne(y2[w + 1]) << 16);
        }
    } else {
#pragma unroll
        for (int w = 0; w < NP; ++w) {
            x1[w] = __float_as_uint(y1[w]);
            x2[w] = __float_as_uint(y2[w]);
        }
    }
    *(u32x4*)(dst + o) = x1;
    *(u32x4*)(dst + o + ho) = x2;
}

template <int DTYPE>
__global__ __launch_bounds__(256) void rope_rows_kernel(RopeRowsParams p) {
    rope_rows_block<DTYPE>(p, blockIdx.x);
}

hipError_t launch_rope_rows(const RopeRowsParams& p, hipStream_t stream) {
    const int np = p.dtype == ADAPSHOT_BF16 ? 8 : 4;
    const int64_t n = (int64_t)p.t_q * p.n_q_heads * (p.head_dim / 2 / np);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (p.dtype == ADAPSHOT_BF16)
        launch_kernel(rope_rows_kernel<ADAPSHOT_BF16>, dim3(blocks), dim3(256), stream, p);
    else
        launch_kernel(rope_rows_kernel<ADAPSHOT_F32>, dim3(blocks), dim3(256), stream, p);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void copy_table_kernel(u32x4_t* dst, const u32x4_t* src, size_t n16) {
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_copy_table(void* dst, const void* src_pinned, size_t bytes, hipStream_t stream) {
    const size_t n16 = bytes / 16;
    if (n16 == 0) return hipSuccess;
    const unsigned blocks = (unsigned)std::min<size_t>((n16 + 255) / 256, 512);
    launch_kernel(copy_table_kernel, dim3(blocks), dim3(256), stream, (u32x4_t*)dst, (const u32x4_t*)src_pinned, n16);
    return hipGetLastError();
}

// ---- plan of a zero-copy context ----------------------------------------------------------
// Blocks 0 .. n_segs-1 expand one shot each into slot_src (context slot -> pool token); the blocks after them
// form tile_rot's row i, (cos, sin)((pos0 + 64 i + 31.5) theta_f), for every 64-slot tile, one fp32 angle addition of the
// two fp64-built table entries.  Where pos0 is a multiple of 64 the addition is that of 0, and a key's angle in the key loop the only rounded
// one: error 3.8e-8 rms (with the centre put together from tab_hi and a half position 5.1e-8).
__global__ __launch_bounds__(256) void pool_plan_kernel(PoolPlanParams p) {
    if ((int)blockIdx.x < p.n_segs) {
        const PoolSeg sg = p.segs[blockIdx.x];
        for (int t = threadIdx.x; t < sg.len; t += 256) p.slot_src[sg.slot0 + t] = sg.src_tok0 + t;
        return;
    }
    const int half = p.head_dim >> 1;
    const int64_t idx = (int64_t)(blockIdx.x - p.n_segs) * 256 + threadIdx.x;
    if (idx >= (int64_t)p.n_tiles * half) return;
    const int64_t tile = idx / half;
    const int f = (int)(idx - tile * half);
    const int64_t a = p.pos0 + tile * 64;
    const float2 h = p.tab_mid[(a >> kRopeLoBits) * half + f], l = p.tab_lo[(a & (kRopeLo - 1)) * half + f];
    p.tile_rot[tile * half + tile_rot_place(f)] = make_float2(h.x * l.x - h.y * l.y, h.y * l.x + h.x * l.y);
}

hipError_t launch_pool_plan(const PoolPlanParams& p, hipStream_t stream) {
    const int64_t rot_blocks = ((int64_t)p.n_tiles * (p.head_dim / 2) + 255) / 256;
    const int64_t blocks = p.n_segs + rot_blocks;
    if (blocks <= 0) return hipSuccess;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    launch_kernel(pool_plan_kernel, dim3((unsigned)blocks), dim3(256), stream, p);
    return hipGetLastError();
}

// ---- combine --------------------------------------------------------------------------------
// out = sum_s 2^(m_s - M) f_s O'_s / sum_s 2^(m_s - M) l_s with M = max_s m_s.  HBM-bound on the partials.
// 16 lanes of 8 fp16 elements (16 bytes per lane) per (kv head, row) pair, so a workgroup of 256 lanes handles 16
// pairs; the partial rows of SB splits are requested together before any is used.  The self split always holds at
// least one visible key, so the denominator is > 0.
template <int SB>
__device__ __forceinline__ void attn_combine_rows(const AttnParams& p, int64_t pair0) {
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    constexpr int d = 128;
    const int g = p.n_q_heads / p.n_kv_heads;
    const int rows = p.t_q * g, n_pairs = rows * p.n_kv_heads;  // (query rows span less than 2 GiB)
    const int pair = (int)pair0 + (int)(threadIdx.x / 16);
    if (pair >= n_pairs) return;
    const int c = threadIdx.x % 16;
    const int hk = (int)((unsigned)pair / (unsigned)rows);
    const int row = pair - hk * rows;
    const int j = (int)((unsigned)row / (unsigned)g);
    const int h = hk * g + (row - j * g);
    const int ns = p.n_split + 1;
    const int64_t split_stride = n_pairs;
    const float4* mlf = p.part_mlf + pair;
    const char* po = (const char*)p.part_o + ((int64_t)pair * d + 8 * c) * 2;

    // One round of loads per SB splits: their (m, l, f) and their rows are requested together; the running
    // maximum M is raised afterwards and what has been accumulated is rescaled (nothing yet: factor 0).
    float M = -INFINITY, L = 0.f;
    f32x8 acc;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    for (int s0 = 0; s0 < ns; s0 += SB) {
        float4 mv[SB];
        f16x8 o[SB];
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const bool on = s0 + u < ns;
            const int64_t so = (int64_t)(s0 + u) * split_stride;
            mv[u] = on ? mlf[so] : make_float4(-INFINITY, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < 8; ++i) o[u][i] = 0;
            if (on) o[u] = __builtin_nontemporal_load((const f16x8*)(po + so * (d * 2)));
        }
        float cm = mv[0].x;
#pragma unroll
        for (int u = 1; u < SB; ++u) cm = fmaxf(cm, mv[u].x);
        const float M_new = fmaxf(M, cm);
        const float r = M == -INFINITY ? 0.f : exp2f(M - M_new);
        M = M_new;
        L *= r;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] *= r;
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const float w = mv[u].x == -INFINITY ? 0.f : exp2f(mv[u].x - M);  // empty or absent split: 0
            L += w * mv[u].y;
            const float wf = w * mv[u].z;
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[i] += wf * (float)o[u][i];
        }
    }
    const float inv = 1.0f / L;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] *= inv;
    *(bf16x8*)((unsigned short*)p.out + ((int64_t)j * p.n_q_heads + h) * d + 8 * c) = __builtin_convertvector(acc, bf16x8);
}

// One kernel per number of splits in flight: it sets the register count (16 partial rows and their (m, l, f) are 128
// registers), and a launch with thousands of workgroups -- the combine of a probe sweep -- lives on how many of them fit
// a compute unit (one kernel for all forms: 244 registers, two wavefronts per SIMD, 40 us for the sweep's 6144
// workgroups).  8 splits in flight when a row has at most 8 partials, else 16.
template <int SB>
__global__ __launch_bounds__(256) void attn_combine_kernel(AttnParams p) {
    attn_combine_rows<SB>(p, (int64_t)blockIdx.x * 16);
}

template <int SB>
__global__ __launch_bounds__(256) void attn_combine_batched_kernel(const AttnBatchItem* items, const CombineWork* work) {
    const CombineWork w = work[blockIdx.x];
    attn_combine_rows<SB>(items[w.item].attn, w.pair0);
}

template <int SB>
__global__ __launch_bounds__(256) void attn_combine_args_kernel(CombineArgs a) {
    const int lane = threadIdx.x & 63;
    const int start = lane < kBatchArgItems ? a.it[lane % kBatchArgItems].block0 : INT32_MAX;
    const int item = __builtin_amdgcn_readfirstlane((int)__popcll(__builtin_amdgcn_ballot_w64(start <= (int)blockIdx.x)) - 1);
    const auto& it = a.it[item];
    AttnParams p;
    p.part_o = (char*)a.part_o + (int64_t)it.part_row0 * 256;
    p.part_mlf = const_cast<float4*>(a.part_mlf) + it.part_row0;
    p.out = it.out;
    p.n_split = it.n_split;
    p.t_q = it.t_q;
    p.n_q_heads = a.n_q_heads;
    p.n_kv_heads = a.n_kv_heads;
    attn_combine_rows<SB>(p, (int64_t)((int)blockIdx.x - it.block0) * 16);
}

hipError_t launch_attn_combine_batch_args(const CombineArgs& a, int n_wgs, int max_partials, hipStream_t stream) {
    if (n_wgs <= 0) return hipSuccess;
    if (max_partials > 8) launch_kernel(attn_combine_args_kernel<16>, dim3((unsigned)n_wgs), dim3(256), stream, a);
    else launch_kernel(attn_combine_args_kernel<8>, dim3((unsigned)n_wgs), dim3(256), stream, a);
    return hipGetLastError();
}

hipError_t launch_attn_combine(const AttnParams& p, hipStream_t stream) {
    const int64_t n_pairs = (int64_t)p.t_q * p.n_q_heads;
    const unsigned blocks = (unsigned)((n_pairs + 15) / 16);
    if (p.n_split + 1 > 8) launch_kernel(attn_combine_kernel<16>, dim3(blocks), dim3(256), stream, p);
    else launch_kernel(attn_combine_kernel<8>, dim3(blocks), dim3(256), stream, p);
    return hipGetLastError();
}

// max_partials is the largest number of partial rows that any item merges per output row.
hipError_t launch_attn_combine_batched(const AttnBatchItem* items, const CombineWork* work, int n_work, int max_partials,
                                       hipStream_t stream) {
    if (n_work <= 0) return hipSuccess;
    if (max_partials > 8) launch_kernel(attn_combine_batched_kernel<16>, dim3((unsigned)n_work), dim3(256), stream, items, work);
    else launch_kernel(attn_combine_batched_kernel<8>, dim3((unsigned)n_work), dim3(256), stream, items, work);
    return hipGetLastError();
}

}  // namespace adapshot
