// Relevance ranking of the pool's shots for a query (Eq. attention_score, Attention-based retrieval): the small
// kernels around the matrix-core pass over the keys (rank_mfma.hip), and the plain kernels of the shapes that pass does
// not cover.
//   rank_prepare   once per pool layer that stores un-rotated keys: every key rotated to its position inside its shot
//                  (Eq. prefill caches them encoded);
//   rank_weights   per (kv head, row): merge the splits' (m, l) into the row's global normaliser and leave
//                  w[s][row] = 2^(m_s - M) / L for every split;
//   rank_reduce    per shot: sum w[split][row] * part[segment][row] over its segments and all rows, always in the same
//                  order (the same query gives the same bits every time), scaled by 1 / (T_q H_q T_i).
#include <algorithm>

#include "mfma_tiles.h"

namespace adapshot {

// grid = (shot, slice of the shot); one thread per (token, kv head, chunk pair): bf16, 8 pairs per 16-byte chunk.
__global__ __launch_bounds__(256) void rank_prepare_kernel(RankPrepareParams p) {
    const int half = p.head_dim >> 1;
    const int cpr = half / 8;  // chunk pairs per head
    const int64_t tok0 = p.shot_off[blockIdx.x];
    const int64_t n = ((int64_t)p.shot_off[blockIdx.x + 1] - tok0) * p.n_kv_heads * cpr;
    for (int64_t idx = (int64_t)blockIdx.y * 256 + threadIdx.x; idx < n; idx += (int64_t)gridDim.y * 256) {
        const int ci = (int)(idx % cpr);
        const int64_t th = idx / cpr;
        const int hk = (int)(th % p.n_kv_heads);
        const int64_t a = th / p.n_kv_heads;  // position inside the shot
        const int64_t o = (((tok0 + a) * p.n_kv_heads + hk) * p.head_dim + ci * 8) * 2;
        const int64_t ho = (int64_t)half * 2;
        const float2* thi = p.tab_hi + (a >> kRopeLoBits) * half + ci * 8;
        const float2* tlo = p.tab_lo + (a & (kRopeLo - 1)) * half + ci * 8;
        u32x4 x1 = *(const u32x4*)(p.k_pool + o), x2 = *(const u32x4*)(p.k_pool + o + ho);
        float y1[8], y2[8];
#pragma unroll
        for (int w = 0; w < 8; ++w) {
            const float2 h = thi[w], l = tlo[w];
            const float c = h.x * l.x - h.y * l.y;
            const float s = h.y * l.x + h.x * l.y;
            const unsigned w1 = x1[w >> 1], w2 = x2[w >> 1];
            const float a1 = (w & 1) ? __uint_as_float(w1 & 0xffff0000u) : __uint_as_float(w1 << 16);
            const float a2 = (w & 1) ? __uint_as_float(w2 & 0xffff0000u) : __uint_as_float(w2 << 16);
            y1[w] = a1 * c - a2 * s;
            y2[w] = a2 * c + a1 * s;
        }
#pragma unroll
        for (int w = 0; w < 8; w += 2) {
            x1[w >> 1] = pack2_bf16(y1[w], y1[w + 1]);
            x2[w >> 1] = pack2_bf16(y2[w], y2[w + 1]);
        }
        *(u32x4*)(p.k_out + o) = x1;
        *(u32x4*)(p.k_out + o + ho) = x2;
    }
}

hipError_t launch_rank_prepare(const RankPrepareParams& p, hipStream_t stream) {
    if (p.n_shots <= 0) return hipSuccess;
    // a slice is 32 tokens of the longest shot, at most 64 slices
    const int64_t slices = std::min<int64_t>(64, std::max<int64_t>(1, (p.max_len + 31) / 32));
    launch_kernel(rank_prepare_kernel, dim3((unsigned)p.n_shots, (unsigned)slices), dim3(256), stream, p);
    return hipGetLastError();
}

// 16 lanes per (kv head, row) pair, lane sl taking splits sl, sl + 16, ...
__global__ __launch_bounds__(256) void rank_weights_kernel(RankReduceParams p) {
    const int sl = threadIdx.x & 15;
    const int64_t pair = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool on = pair < p.n_pairs;  // whole 16-lane groups are on or off together
    float M = -INFINITY;
    if (on)
        for (int s = sl; s < p.n_split; s += 16) M = fmaxf(M, p.part_ml[(int64_t)s * p.n_pairs + pair].x);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) M = fmaxf(M, __shfl_xor(M, o, 64));
    float L = 0.f;
    if (on)
        for (int s = sl; s < p.n_split; s += 16) {
            const float2 v = p.part_ml[(int64_t)s * p.n_pairs + pair];
            L += exp2f(v.x - M) * v.y;
        }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) L += __shfl_xor(L, o, 64);
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    if (on)
        for (int s = sl; s < p.n_split; s += 16)
            p.weights[(int64_t)s * p.n_pairs + pair] = exp2f(p.part_ml[(int64_t)s * p.n_pairs + pair].x - M) * inv;
}

// One workgroup per shot.  VEC: whole 16-byte pieces (the number of pairs is a multiple of 4).
template <bool VEC>
__global__ __launch_bounds__(256) void rank_reduce_kernel(RankReduceParams p) {
    __shared__ float red[4];
    const int i = blockIdx.x;
    float acc = 0.f;
    for (int q = p.shot_seg0[i]; q < p.shot_seg0[i + 1]; ++q) {
        const float* v = p.part + (int64_t)q * p.n_pairs;
        const float* w = p.weights + (int64_t)p.seg_split[q] * p.n_pairs;
        if (VEC) {
#pragma unroll 4
            for (int64_t r = threadIdx.x * 4; r < p.n_pairs; r += 1024) {
                const f32x4 a = __builtin_nontemporal_load((const f32x4*)(v + r)), b = *(const f32x4*)(w + r);
                acc += (a[0] * b[0] + a[1] * b[1]) + (a[2] * b[2] + a[3] * b[3]);
            }
        } else {
            for (int64_t r = threadIdx.x; r < p.n_pairs; r += 256) acc += v[r] * w[r];
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) p.scores[i] = ((red[0] + red[1]) + (red[2] + red[3])) * p.inv_rows * p.inv_len[i];
}

hipError_t launch_rank_weights(const RankReduceParams& p, hipStream_t stream) {
    if (p.n_split <= 0 || p.n_pairs <= 0) return hipSuccess;
    launch_kernel(rank_weights_kernel, dim3((unsigned)((p.n_pairs + 15) / 16)), dim3(256), stream, p);
    return hipGetLastError();
}

hipError_t launch_rank_reduce(const RankReduceParams& p, hipStream_t stream) {
    if (p.n_pairs <= 0 || p.n_shots <= 0) return hipSuccess;
    if (p.n_pairs % 4 == 0) launch_kernel(rank_reduce_kernel<true>, dim3((unsigned)p.n_shots), dim3(256), stream, p);
    else launch_kernel(rank_reduce_kernel<false>, dim3((unsigned)p.n_shots), dim3(256), stream, p);
    return hipGetLastError();
}

// ---- shapes the matrix-core kernel does not cover ------------------------------------------------------
template <int DTYPE>
__device__ __forceinline__ float rank_load(const void* base, int64_t i) {
    if (DTYPE == ADAPSHOT_BF16) return __uint_as_float(((unsigned)((const unsigned short*)base)[i]) << 16);
    return ((const float*)base)[i];
}
__device__ __forceinline__ float rank_wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float rank_wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// One wavefront per (query token j, head h).  score(u) = q~ . k~_u in log2 units, k~_u = the key of pool token u
// as a cache holds it: encoded at its position inside its shot and rounded to the storage type (a pool that
// stores un-rotated keys), or as stored.  Pass 1: the row's maximum and sum over the whole pool; pass 2: the
// normalised mass of every shot.
template <int DTYPE>
__global__ __launch_bounds__(64) void rank_generic_kernel(RankGenericParams p) {
    __shared__ float q_s[1024];
    const int lane = threadIdx.x;
    const int d = p.head_dim, half = d >> 1;
    const int g = p.n_q_heads / p.n_kv_heads;
    const int r = blockIdx.x;  // j * h_q + h
    const int h = r % p.n_q_heads;
    const int hk = h / g;
    for (int e = lane; e < d; e += 64) q_s[e] = rank_load<DTYPE>(p.q_rot, (int64_t)r * d + e);
    __syncthreads();
    auto score = [&](int64_t u, int64_t t_local) -> float {
        const int64_t o = (u * p.n_kv_heads + hk) * d;
        float dot = 0.f;
        if (p.key_state == ADAPSHOT_KEYS_UNROTATED) {
            const float2* th = p.tab_hi + (t_local >> kRopeLoBits) * half;
            const float2* tl = p.tab_lo + (t_local & (kRopeLo - 1)) * half;
            for (int i = 0; i < half; ++i) {
                const float2 hh = th[i], ll = tl[i];
                const float c = hh.x * ll.x - hh.y * ll.y, sn = hh.y * ll.x + hh.x * ll.y;
                const float x1 = rank_load<DTYPE>(p.k_pool, o + i), x2 = rank_load<DTYPE>(p.k_pool, o + i + half);
                float y1 = x1 * c - x2 * sn, y2 = x2 * c + x1 * sn;
                if (DTYPE == ADAPSHOT_BF16) {
                    y1 = __uint_as_float((unsigned)__builtin_bit_cast(unsigned short, (__bf16)y1) << 16);
                    y2 = __uint_as_float((unsigned)__builtin_bit_cast(unsigned short, (__bf16)y2) << 16);
                }
                dot += q_s[i] * y1 + q_s[i + half] * y2;
            }
        } else {
            for (int e = 0; e < d; ++e) dot += q_s[e] * rank_load<DTYPE>(p.k_pool, o + e);
        }
        return dot;
    };
    float m = -INFINITY, l = 0.f;  // per lane; merged below
    for (int i = 0; i < p.n_shots; ++i) {
        const int64_t t0 = p.shot_off[i], t1 = p.shot_off[i + 1];
        for (int64_t u = t0 + lane; u < t1; u += 64) {
            const float s = score(u, u - t0);
            const float mn = fmaxf(m, s);
            l = l * exp2f(m - mn) + exp2f(s - mn);
            m = mn;
        }
    }
    const float M = rank_wave_max(m);
    const float L = rank_wave_sum(m == -INFINITY ? 0.f : l * exp2f(m - M));
    const float inv_l = 1.0f / L;
    for (int i = 0; i < p.n_shots; ++i) {
        const int64_t t0 = p.shot_off[i], t1 = p.shot_off[i + 1];
        float a = 0.f;
        for (int64_t u = t0 + lane; u < t1; u += 64) a += exp2f(score(u, u - t0) - M);
        a = rank_wave_sum(a);
        if (lane == 0) p.mass[(int64_t)r * p.n_shots + i] = a * inv_l;
    }
}

// One thread per shot: the rows' masses added in row order, scaled by 1 / (T_q H_q T_i).
__global__ __launch_bounds__(256) void rank_generic_finish_kernel(RankGenericParams p) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= p.n_shots) return;
    const int n_rows = p.t_q * p.n_q_heads;
    float a = 0.f;
    for (int r = 0; r < n_rows; ++r) a += p.mass[(int64_t)r * p.n_shots + i];
    const float len = (float)(p.shot_off[i + 1] - p.shot_off[i]);
    p.scores[i] = a / ((float)n_rows * len);
}

hipError_t launch_rank_generic(const RankGenericParams& p, hipStream_t stream) {
    if (p.head_dim > 1024) return hipErrorInvalidValue;
    const unsigned rows = (unsigned)(p.t_q * p.n_q_heads);
    if (p.dtype == ADAPSHOT_BF16)
        launch_kernel(rank_generic_kernel<ADAPSHOT_BF16>, dim3(rows), dim3(64), stream, p);
    else
        launch_kernel(rank_generic_kernel<ADAPSHOT_F32>, dim3(rows), dim3(64), stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    launch_kernel(rank_generic_finish_kernel, dim3((unsigned)((p.n_shots + 255) / 256)), dim3(256), stream, p);
    return hipGetLastError();
}

}  // namespace adapshot
