// Entropy of softmax(logits) over the whole vocabulary (Eq. entropy), natural log.
//
// With m = max z, e_v = exp(z_v - m), s = sum e_v, t = sum (z_v - m) e_v:
//     H = ln s - t / s.
// One HBM pass: a workgroup reduces one chunk of one row to (m, s, t) with an online
// rescale per 16-element batch; the workgroup that arrives last merges the chunks of its row.
// Partials re-base as  s' = s * exp(m - M),  t' = (t + (m - M) * s) * exp(m - M).
#include <mutex>

#include "mfma_tiles.h"

namespace adapshot {


// Chunk partials of the entry point that allocates nothing: kStaticEntropyPartials (row, chunk) triples,
// 768 KiB, held by every GPU the library runs on until the process ends.  Host code never uses this name as
// an address: entropy_static_scratch() asks the runtime where the current device keeps its copy.
static __device__ __align__(256) float g_entropy_scratch[(size_t)kStaticEntropyPartials * 3];

hipError_t entropy_static_scratch(float** out) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static float* ptr_of_device[kMaxDevices] = {};
    *out = nullptr;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of_device[dev]) {  // once per device, with that device current
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(g_entropy_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptr_of_device[dev] = (float*)p;
    }
    *out = ptr_of_device[dev];
    return hipSuccess;
}

struct Mst {
    float m, s, t;
};

// Merge b into a.  -inf maxima (empty parts) are handled by the w == 0 branches.
__device__ __forceinline__ Mst mst_merge(Mst a, Mst b) {
    const float M = fmaxf(a.m, b.m);
    Mst r;
    r.m = M;
    if (M == -INFINITY) {  // both empty so far (or all -inf): keep sums as they are (0, or NaN markers)
        r.s = a.s + b.s;
        r.t = a.t + b.t;
        return r;
    }
    const float da = a.m - M, db = b.m - M;  // <= 0, may be -inf
    const float wa = __expf(da), wb = __expf(db);
    const float ta = wa > 0.f ? (a.t + da * a.s) * wa : 0.f;
    const float tb = wb > 0.f ? (b.t + db * b.s) * wb : 0.f;
    r.s = a.s * wa + b.s * wb;
    r.t = ta + tb;
    return r;
}

// The 64 lanes' parts merged, in every lane: the largest maximum first, each lane re-based to it once, then two plain sums (lane
// by lane in six rounds of mst_merge, two exponentials and three exchanges through LDS each, took 1 us).
__device__ __forceinline__ Mst mst_wave_reduce(Mst v) {
    const float M = wave_max(v.m);  // a maximum is never NaN (fmaxf)
    if (M != -INFINITY) {  // the same for all lanes; else all empty, or nothing but -inf: sums as they are
        const float d = v.m - M;
        const float w = __expf(d);
        v.t = w > 0.f ? (v.t + d * v.s) * w : 0.f;
        v.s *= w;
    }
    return Mst{M, wave_sum(v.s), wave_sum(v.t)};
}

// a * b with 0 * anything = 0 (v_mul_legacy_f32)
__device__ __forceinline__ float mul_legacy(float a, float b) {
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// Fold a batch of N values into the running (m, s, t).  A NaN logit poisons s through exp(NaN); a -inf
// logit gives e = 0 and must contribute 0 to t although dz = -inf: the legacy multiply returns 0 for
// 0 * anything, which is exactly the limit p ln p -> 0.
template <int N>
__device__ __forceinline__ void mst_add_batch(Mst& acc, const float (&z)[N]) {
    float bm = z[0];
#pragma unroll
    for (int i = 1; i < N; ++i) bm = fmaxf(bm, z[i]);
    const float M = fmaxf(acc.m, bm);
    if (M == INFINITY) {  // +inf logit: the row has no distribution
        acc.m = M;
        acc.s = NAN;
        acc.t = NAN;
        return;
    }
    if (M == -INFINITY) {  // nothing but -inf so far, unless a NaN hides behind the maximum (fmaxf skips NaN)
        bool nan = false;
#pragma unroll
        for (int i = 0; i < N; ++i) nan |= (z[i] != z[i]);
        if (nan) {
            acc.s = NAN;
            acc.t = NAN;
        }
        return;
    }
    if (M > acc.m) {
        const float dm = acc.m - M;
        const float w = __expf(dm);  // acc.m = -inf -> 0
        acc.t = w > 0.f ? (acc.t + dm * acc.s) * w : 0.f;
        acc.s *= w;
        acc.m = M;
    }
    float s = 0.f, t = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float dz = z[i] - M;
        const float e = __expf(dz);
        s += e;
        t += mul_legacy(e, dz);
    }
    acc.s += s;
    acc.t += t;
}

// (m, s, t) of one chunk of a row, by 256 threads; the result is thread 0's.  VEC: rows are 16-byte aligned -> float4 loads.
template <bool VEC>
__device__ __forceinline__ Mst reduce_chunk(const EntropyParams& p, int row, int chunk) {
    __shared__ Mst red[4];
    const int tid = threadIdx.x;
    const float* z = p.logits + (int64_t)row * p.row_stride;
    const int c0 = chunk * p.chunk;
    const int c1 = min(c0 + p.chunk, p.vocab);
    Mst acc = {-INFINITY, 0.f, 0.f};
    if (VEC) {
        // 4 float4 per thread per step, each load instruction covering 4 KB contiguous per workgroup.  Full
        // steps (the common case) take a branch-free path and the next step's loads are issued before this
        // step's values are used; the ragged last step of a row checks every element.
        auto load_full = [&](int base, float (&v)[16]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4 x = __builtin_nontemporal_load((const f32x4*)(z + base + u * 1024 + tid * 4));
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * u + k] = x[k];
            }
        };
        int base = c0;
        if (base + 4096 <= c1) {
            float cur[16];
            load_full(base, cur);
            base += 4096;
            while (base + 4096 <= c1) {
                float nxt[16];
                load_full(base, nxt);
                base += 4096;
                mst_add_batch<16>(acc, cur);
#pragma unroll
                for (int k = 0; k < 16; ++k) cur[k] = nxt[k];
            }
            mst_add_batch<16>(acc, cur);
        }
        for (; base < c1; base += 4096) {
            float v[16];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + u * 1024 + tid * 4;
                f32x4 x = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                if (i + 3 < c1) {
                    x = __builtin_nontemporal_load((const f32x4*)(z + i));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (i + k < c1) x[k] = z[i + k];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * u + k] = x[k];
            }
            mst_add_batch<16>(acc, v);
        }
    } else {
        for (int base = c0; base < c1; base += 1024) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + u * 256 + tid;
                v[u] = i < c1 ? z[i] : -INFINITY;
            }
            mst_add_batch<4>(acc, v);
        }
    }
    acc = mst_wave_reduce(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    return mst_merge(mst_merge(red[0], red[1]), mst_merge(red[2], red[3]));
}

// The entropy of a row from its (m, s, t), by one wavefront (all lanes hold r).  TOKENS: Eq. (entropy) as printed, summed over
// the answer tokens C only; lane c < |C| holds token c.
//   full-p reading:      H = -sum_c p_c ln p_c,  ln p_c = z_c - lse
//   renormalised reading: the same with the log-sum-exp taken over C
// A term with p_c = 0 contributes 0.
template <bool TOKENS>
__device__ __forceinline__ void finish_row(const EntropyParams& p, const AnswerTokens& c, int row, Mst r, int lane) {
    if (!TOKENS) {
        if (lane == 0) {
            float h;
            if (r.m == -INFINITY || r.m == INFINITY) h = NAN;  // no finite logit, or a +inf logit
            else h = logf(r.s) - r.t / r.s;                   // NaN sums propagate
            p.out[row] = h;
        }
        return;
    }
    const bool row_bad = r.m == -INFINITY || r.m == INFINITY || r.s != r.s;  // as in the full entropy
    const float zc = lane < c.n ? p.logits[(int64_t)row * p.row_stride + c.id[lane]] : -INFINITY;
    float lse;
    if (c.mode == ADAPSHOT_ENTROPY_FULL_P) {
        lse = r.m + logf(r.s);
    } else {
        float mc = zc;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) mc = fmaxf(mc, __shfl_xor(mc, o, 64));
        float sc = mc == -INFINITY ? 0.f : expf(zc - mc);  // lanes past |C| hold -inf: 0
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sc += __shfl_xor(sc, o, 64);
        lse = mc + logf(sc);
        if (mc == -INFINITY) lse = NAN;  // all of C at -inf
    }
    const float lp = zc - lse;
    const float pc = expf(lp);
    float h = (lane < c.n && pc > 0.f) ? -pc * lp : 0.f;
    if (lse != lse) h = NAN;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) h += __shfl_xor(h, o, 64);
    if (lane == 0) p.out[row] = row_bad ? NAN : h;
}

// grid = n_rows * n_chunks workgroups (chunk fastest), 256 threads.
template <bool VEC>
__global__ __launch_bounds__(256) void entropy_chunk_kernel(EntropyParams p) {
    const int row = blockIdx.x / p.n_chunks;
    const Mst r = reduce_chunk<VEC>(p, row, blockIdx.x - row * p.n_chunks);
    if (threadIdx.x == 0) {
        float* o = p.partials + (int64_t)blockIdx.x * 3;
        o[0] = r.m;
        o[1] = r.s;
        o[2] = r.t;
    }
}

// The same, and the workgroup that arrives last at its row's counter merges the row's chunks (in chunk order, whatever the
// order of arrival): one launch.  Partials go past the L2 of the workgroup's XCD and are waited for before the arrival, so
// no cache is written back or invalidated; the counter is zero again afterwards.  What it has to avoid is counters that
// share a line (counter_stride).  Kernel time over logits that no cache holds, with chunks of 1024 to 8192 floats and a merge by
// exchanges / with 4096 and 8192 and one re-base per lane (us): 1 row of 128256 6.8 / 4.8, 16 rows 9.7 / 5.8, 48 rows 8.9 / 7.6, 128
// rows 15.0 / 13.6 (4.8 TB/s), 200 rows 20.6 / 19.4; 8 rows of 50257 5.7 / 4.3.  Two launches take 3 us more up to 48 rows.
template <bool VEC, bool TOKENS>
__global__ __launch_bounds__(256) void entropy_fused_kernel(EntropyParams p, AnswerTokens c) {
    __shared__ int last_flag;
    const int tid = threadIdx.x;
    const int row = blockIdx.x / p.n_chunks;
    Mst r = reduce_chunk<VEC>(p, row, blockIdx.x - row * p.n_chunks);  // the same in every thread
    if (p.n_chunks > 1) {
        if (tid == 0) {
            float* o = p.partials + (int64_t)blockIdx.x * 3;
            __hip_atomic_store(o, r.m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 1, r.s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(o + 2, r.t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the partial has reached memory
            const unsigned before = __hip_atomic_fetch_add(p.counters + row * p.counter_stride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const bool mine = before == (unsigned)p.n_chunks - 1u;
            if (mine) __hip_atomic_store(p.counters + row * p.counter_stride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last_flag = mine ? 1 : 0;
        }
        __syncthreads();
        if (!last_flag) return;
        if (tid >= 64) return;
        r = Mst{-INFINITY, 0.f, 0.f};
        for (int k = tid; k < p.n_chunks; k += 64) {
            const float* o = p.partials + ((int64_t)row * p.n_chunks + k) * 3;
            Mst b;
            b.m = __hip_atomic_load(o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            b.s = __hip_atomic_load(o + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            b.t = __hip_atomic_load(o + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r = mst_merge(r, b);
        }
        r = mst_wave_reduce(r);
    }
    if (tid < 64) finish_row<TOKENS>(p, c, row, r, tid);
}

// Whole rows in one launch: a workgroup of 1024 threads reduces one row and writes its entropy (or, with answer
// tokens, Eq. (entropy) over those) itself.  The same per-thread stream and merge as the chunk kernel; used when
// there are enough rows to keep the memory system busy with one workgroup per row, which saves the second launch.
template <bool VEC, bool TOKENS>
__global__ __launch_bounds__(1024) void entropy_row_kernel(EntropyParams p, AnswerTokens c) {
    __shared__ Mst red[16];
    const int tid = threadIdx.x;
    const int row = blockIdx.x;
    const float* z = p.logits + (int64_t)row * p.row_stride;
    const int c1 = p.vocab;
    Mst acc = {-INFINITY, 0.f, 0.f};
    if (VEC) {
        auto load_full = [&](int base, float (&v)[16]) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const f32x4 x = __builtin_nontemporal_load((const f32x4*)(z + base + u * 4096 + tid * 4));
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * u + k] = x[k];
            }
        };
        // one step (16384 logits) ahead; more in flight does not help a lone workgroup (a compute unit alone sustains
        // about 40 GB/s: 12.8 us for a 513 KB row, 14.5 us with three steps in flight)
        int base = 0;
        if (base + 16384 <= c1) {
            float cur[16];
            load_full(base, cur);
            base += 16384;
            while (base + 16384 <= c1) {
                float nxt[16];
                load_full(base, nxt);
                base += 16384;
                mst_add_batch<16>(acc, cur);
#pragma unroll
                for (int k = 0; k < 16; ++k) cur[k] = nxt[k];
            }
            mst_add_batch<16>(acc, cur);
        }
        for (; base < c1; base += 16384) {
            float v[16];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + u * 4096 + tid * 4;
                f32x4 x = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                if (i + 3 < c1) {
                    x = __builtin_nontemporal_load((const f32x4*)(z + i));
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (i + k < c1) x[k] = z[i + k];
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) v[4 * u + k] = x[k];
            }
            mst_add_batch<16>(acc, v);
        }
    } else {
        for (int base = 0; base < c1; base += 4096) {
            float v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = base + u * 1024 + tid;
                v[u] = i < c1 ? z[i] : -INFINITY;
            }
            mst_add_batch<4>(acc, v);
        }
    }
    acc = mst_wave_reduce(acc);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid >= 64) return;
    const int lane = tid;
    Mst r = {-INFINITY, 0.f, 0.f};
    if (lane < 16) r = red[lane];
    r = mst_wave_reduce(r);
    finish_row<TOKENS>(p, c, row, r, lane);
}

hipError_t launch_entropy_rows(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream) {
    const bool vec = entropy_rows_aligned(p.logits, p.row_stride);
    const dim3 grid((unsigned)p.n_rows);
    const AnswerTokens none{};
    if (c) {
        if (vec) launch_kernel((entropy_row_kernel<true, true>), grid, dim3(1024), stream, p, *c);
        else launch_kernel((entropy_row_kernel<false, true>), grid, dim3(1024), stream, p, *c);
    } else {
        if (vec) launch_kernel((entropy_row_kernel<true, false>), grid, dim3(1024), stream, p, none);
        else launch_kernel((entropy_row_kernel<false, false>), grid, dim3(1024), stream, p, none);
    }
    return hipGetLastError();
}

// One wavefront per row merges its chunk partials and writes H: calls of many rows, and the entry point that has no counters.
template <bool TOKENS>
__global__ __launch_bounds__(64) void entropy_finish_kernel(EntropyParams p, AnswerTokens c) {
    const int row = blockIdx.x;
    const int lane = threadIdx.x;
    Mst acc = {-INFINITY, 0.f, 0.f};
    for (int k = lane; k < p.n_chunks; k += 64) {
        const float* o = p.partials + ((int64_t)row * p.n_chunks + k) * 3;
        Mst b = {o[0], o[1], o[2]};
        acc = mst_merge(acc, b);
    }
    acc = mst_wave_reduce(acc);
    finish_row<TOKENS>(p, c, row, acc, lane);
}

hipError_t launch_entropy_fused(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream) {
    if ((int64_t)p.n_chunks * p.n_rows > INT32_MAX) return hipErrorInvalidValue;  // the host checks this first
    const bool vec = entropy_rows_aligned(p.logits, p.row_stride);
    const dim3 grid((unsigned)(p.n_chunks * p.n_rows)), block(256);
    const AnswerTokens none{};
    if (c) {
        if (vec) launch_kernel((entropy_fused_kernel<true, true>), grid, block, stream, p, *c);
        else launch_kernel((entropy_fused_kernel<false, true>), grid, block, stream, p, *c);
    } else {
        if (vec) launch_kernel((entropy_fused_kernel<true, false>), grid, block, stream, p, none);
        else launch_kernel((entropy_fused_kernel<false, false>), grid, block, stream, p, none);
    }
    return hipGetLastError();
}

hipError_t launch_entropy_chunk(const EntropyParams& p, hipStream_t stream) {
    if ((int64_t)p.n_chunks * p.n_rows > INT32_MAX) return hipErrorInvalidValue;  // the host checks this first
    dim3 grid((unsigned)((int64_t)p.n_chunks * p.n_rows));
    const bool vec = entropy_rows_aligned(p.logits, p.row_stride);
    if (vec)
        launch_kernel(entropy_chunk_kernel<true>, grid, dim3(256), stream, p);
    else
        launch_kernel(entropy_chunk_kernel<false>, grid, dim3(256), stream, p);
    return hipGetLastError();
}

hipError_t launch_entropy_finish(const EntropyParams& p, const AnswerTokens* c, hipStream_t stream) {
    if (c) launch_kernel(entropy_finish_kernel<true>, dim3((unsigned)p.n_rows), dim3(64), stream, p, *c);
    else launch_kernel(entropy_finish_kernel<false>, dim3((unsigned)p.n_rows), dim3(64), stream, p, AnswerTokens{});
    return hipGetLastError();
}

}  // namespace adapshot
