// Query-over-cache attention straight from registers: the kernel for the shapes that the 256-row tile kernel
// (attn_mfma.hip) does not cover -- fp32 models, head dimensions other than 128 -- and for its smaller problems: decode steps and
// probes over contexts of up to a few thousand slots, which would leave most of that kernel's wavefronts without rows and pay
// its second launch (attn_plan.h has the border).
//
// A workgroup of 8 wavefronts owns 16 * NR query rows of one KV head (rows j*g + h%g, as everywhere) and one split of
// the context; the last split also takes the query's own tokens (causal).  The keys go to the wavefronts in steps of 16
// (bf16 models: 32), round robin, and every wavefront runs a flash-attention state of its own over its keys: no
// barrier and no other wavefront in the key loop.  V rows are loaded from global memory in exactly the lanes where
// the matrix instructions want them, K rows whole into LDS and from there into the lanes (or, where that is no gain, straight into them),
// so the loop is loads, matrix instructions and a softmax of 4 or 8 values:
//
//   S^T = K . Q^T   A = K: lane (key l%16, group l/16) holds KW consecutive columns 4*KW*j + KW*(l/16) of its key for
//                   every j (16 bytes), B = Q in the same lanes and columns: bf16 models v_mfma_f32_16x16x32_bf16 on the
//                   stored operands, fp32 models v_mfma_f32_16x16x4_f32.  The result leaves lane l with query row l%16
//                   and keys 4*(l/16) .. +3 of every 16.
//   O^T += V^T.P^T  A lane loads the V rows of just those keys, VW consecutive columns each (a row-wise load of 16 lanes);
//                   the 16 columns of MFMA block (dg, c) are 16*VW*dg + VW*i + c.  fp32 models: v_mfma_f32_16x16x4_f32,
//                   register r of S^T as it stands.  bf16 models: v_mfma_f32_16x16x32_bf16, column c of a lane's 8 rows
//                   picked together by byte permutes, and P in three bf16 pieces -- the upper 8 of its 24 bits, the
//                   next 8, the last 8, exactly -- so that P is not rounded: three instructions of 16 cycles for 32 keys
//                   where the fp32 product took eight of 32.  Head dimension 128 takes two, the second one rounded: 2^-17
//                   of a weight (against float64, 64 query tokens over 830 slots, rel. error of a bf16 result: one rounded
//                   piece 2.8e-3, as in the tile kernel, 2.4e-3 with two, at 2 % more time).
//
// The wavefronts' states meet in LDS once, at the end.  With one split the workgroup writes the output rows itself:
// rotation, attention and merge are then one launch.  With more, each workgroup leaves its merged rows (fp32) and (m, l)
// in a workspace, and the workgroup that arrives last at the unit's counter merges them: partials are written and read
// with device-scope accesses that bypass the L2 of the workgroup's XCD, so no cache has to be written back or invalidated,
// and the counter is back at zero afterwards.  The merge runs in split order whatever the order of arrival: the same
// inputs give the same bits.
//
// What bounds it: a small problem, the launch, two or three round trips to memory (keys and query rows, arrival, partials)
// and the instructions between them, 4 cycles each and two wavefronts per SIMD: loads therefore go through buffers (no
// address arithmetic) and the query rows are rotated once per workgroup and handed out through LDS.  A larger problem,
// what a compute unit gets from beyond its L1 -- 54 KB/us where few of them ask, 45 in launches that fill the chip, whatever is in flight
// (64 or 128 KB) -- which is why the loads are shared by two row blocks where there are rows enough.  Splits beyond a few dozen
// are bound by their merge, which one compute unit does.  One layer, call after call over contexts
// that no cache holds, addresses by lane and splits priced with a warm cache / now
//   bf16, 28/4 heads x 128, one token over 16k slots               19.9 / 13.4 us
//   bf16, 32/8 heads x 128, one token over 4k slots                14.3 / 8.8
//   fp32, 8/2 heads x 128, 32 query tokens over 2k slots           18.7 / 11.7
//   bf16, 32/8 heads x 128, 24 query tokens over 830 slots, tile kernel and its merge 15.5, here 8.5
#pragma once
#include <type_traits>

#include "mfma_tiles.h"

namespace adapshot {

typedef unsigned long long u64;

__device__ __forceinline__ void stream_store2(float* p, float a, float b) {
    const u64 v = (u64)__float_as_uint(a) | ((u64)__float_as_uint(b) << 32);
    __hip_atomic_store((u64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int DTYPE, int D, int NR, bool POOL, int NI>
__global__ __launch_bounds__(kStreamWaves * 64) void attn_stream_kernel(StreamArgs<NI> p) {
    constexpr int W = kStreamWaves, T = W * 64;
    constexpr bool BF = DTYPE == ADAPSHOT_BF16;
    constexpr int E = BF ? 2 : 4;
    constexpr int KW = D * E >= 64 ? 16 / E : D / 4;  // consecutive columns of a lane
    constexpr int NJ = D / (4 * KW);
    constexpr int KR = KW * E / 4;                    // registers of one j
    constexpr int KP = 16 / E;                        // elements of a 16-byte chunk
    constexpr int DB = D >= 16 ? D / 16 : 1;          // 16-column blocks of the output
    constexpr int VMAX = 16 / E;
    constexpr int VW = DB < VMAX ? DB : VMAX;         // consecutive V columns of a lane
    constexpr int DG = DB / VW;
    constexpr int VR = VW * E >= 4 ? VW * E / 4 : 1;  // registers of one V piece
    constexpr int NK = BF && D <= 128 ? 2 : 1;        // 16-key blocks of a step
    constexpr int SK = 16 * NK;                       // keys of a step
    constexpr int NV = 4 * NK;                        // V rows of a lane
    constexpr int NP = BF ? (D == 128 ? 2 : 3) : 0;   // bf16 pieces of a softmax weight (fp32 models: as it is)
    constexpr int STEP_REGS = NJ * KR + 4 * DG * VR;
    // The next step's K and V are loaded while this one is computed (two steps ahead is no faster and costs 16 to 32
    // registers); a step of 256 bytes per lane, or two row blocks over gathered keys, leave room for K alone, V is then loaded
    // under the first product.
    constexpr int NB = 2;
    constexpr int NBV = STEP_REGS > (BF ? 48 : 32) || (BF && POOL && NR == 2) ? 1 : 2;
    // Gathered keys are turned to their positions before the next step's rows are requested, unless V is loaded late, for want of registers:
    // then behind them (bf16 x 256, 64 tokens over 25k slots: before 381 us and 106 registers in memory, behind 206 and 11).
    constexpr bool LATE = POOL && NBV == 1;
    constexpr int TR = 16 * NR;
    constexpr int NS = NR * DB;  // 1 KB pieces of a wavefront's output state
    static_assert(D == 8 || D % 16 == 0, "head dimensions");
    // Keys of an assembled context come through LDS (dma_k), two steps per wavefront, in bf16 models where these and the states fit: the loads are
    // what the loop waits for.  Calls over contexts that no cache held, straight into the lanes / through LDS, us: bf16 x 64, 64 tokens over
    // 6.6k slots 22.3 / 19.5, 32/8 heads x 128, 24 tokens over 830 10.3 / 9.7.  Not fp32, whose matrix instructions take longer than its loads:
    // x 128, 32 tokens over 2k 13.5 / 13.7, x 64, 100 tokens of 32/8 heads over 24k 214 / 222, 16 over 24k 32.5 / 33.1, one of 4/2 over 154 4.7 / 4.5, 16 over 224 6.6 / 6.1.
    constexpr int RB = D * E;                                        // bytes of a row
    constexpr int KS_BYTES = SK * RB;                                // keys of a step
    constexpr int OS_BYTES = NS * 1024 > KS_BYTES ? NS * 1024 : KS_BYTES;
    constexpr bool KL = BF && !POOL && RB >= 128 && W * (OS_BYTES + KS_BYTES) <= 128 * 1024;
    constexpr int RI = KL ? 1024 / RB : 1;                           // rows of one load instruction
    constexpr int CR = RB >= 16 ? RB / 16 : 1;                       // 16-byte chunks of a row
    constexpr int RG = RB < 256 ? 256 / RB : 1, CM = CR < 16 ? CR - 1 : 15;  // row r keeps chunk c at place c ^ (r / RG & CM)

    // (the states take the place of the even steps' keys)
    __shared__ __attribute__((aligned(1024))) char ks0[W * (KL ? OS_BYTES : NS * 1024)];
    __shared__ __attribute__((aligned(1024))) char ks1[KL ? W * KS_BYTES : 16];
    f32x4 (*const os)[NS][64] = (f32x4 (*)[NS][64])ks0;
    __shared__ float2 wml[W][TR];
    __shared__ __attribute__((aligned(16))) char qs[TR * D * E];
    __shared__ float sw[kStreamMaxSplits][TR];
    __shared__ int last_flag;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, kg = lane >> 4;

    // The workgroups of the problems one after the other, none of them empty: empty ones, of the problems with fewer splits, would take
    // turns with the others, and a launch of 256 had two on some compute units (4 queries of 8k slots, 28/4 heads 28 us, 19 without).
    int item = 0;
    if (NI > 1) {
        const int start = lane < NI ? p.it[lane % NI].block0 : INT32_MAX;
        item = __builtin_amdgcn_readfirstlane((int)__popcll(__builtin_amdgcn_ballot_w64(start <= (int)blockIdx.x)) - 1);
    }
    const StreamItem& it = p.it[item];
    const int block = (int)blockIdx.x - (NI > 1 ? it.block0 : 0);
    const int n_split = it.n_split;
    const int hkv = p.n_kv_heads, g = p.g;
    const int rows = it.t_q * g;
    const int rest = p.div_hkv.of(block), hk = block - rest * hkv;
    const int rt = it.div_split.of(rest), split = rest - rt * n_split;
    const int row0 = rt * TR;
    if (row0 >= rows) return;
    const bool last_split = split == n_split - 1;

    const int64_t stride = (int64_t)hkv * D * E;
    const int k0 = split * it.keys_per_split;
    int nk = it.n_ctx - k0;  // context keys of this split
    if (nk > it.keys_per_split) nk = it.keys_per_split;
    if (nk < 0) nk = 0;
    const int j_last = p.div_g.of((row0 + TR < rows ? row0 + TR : rows) - 1);
    const int n_self = last_split ? j_last + 1 : 0;  // own tokens that any row of the tile sees
    const int n_cs = (nk + SK - 1) / SK;
    const int n_steps = n_cs + (n_self + SK - 1) / SK;

    const char* const kself = it.k_self + (int64_t)hk * D * E;
    const char* const vself = it.v_self + (int64_t)hk * D * E;
    const char* const kctx = it.k_ctx + (int64_t)hk * D * E + (POOL ? 0 : k0 * stride);
    const char* const vctx = it.v_ctx + (int64_t)hk * D * E + (POOL ? 0 : k0 * stride);

    // ---- loads of step s.  Steps past the end read no rows (the zero-copy form: one row again, all lanes the same bytes).
    // Zero-copy form: pool tokens of the rows of the next step to load, and (next) of the one after it.  These are requested ahead of
    // the rows of the step before theirs: loads return in order, and behind those rows they would be waited for with them.
    // (Where registers are short they are requested behind them, or, if V is loaded that late, ahead of their own.)
    constexpr bool TOK2 = NBV > 1 && NR == 1;
    int tok_k[NK] = {}, tok_v[NV] = {}, next_k[NK] = {}, next_v[NV] = {};
    auto pool_tok = [&](int u) __attribute__((always_inline)) -> int {
        u = u < nk ? u : nk - 1;
        u = u > 0 ? u : 0;
        return p.slot_src[k0 + u];
    };
    auto fetch_tok = [&](int s) __attribute__((always_inline)) {
        if (POOL && nk > 0) {
#pragma unroll
            for (int b = 0; b < NK; ++b) next_k[b] = pool_tok(SK * s + 16 * b + l16);
#pragma unroll
            for (int r = 0; r < NV; ++r) next_v[r] = pool_tok(SK * s + 16 * (r >> 2) + 4 * kg + (r & 3));
        }
    };
    auto take_tok = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NK; ++b) tok_k[b] = next_k[b];
#pragma unroll
        for (int r = 0; r < NV; ++r) tok_v[r] = next_v[r];
    };
    // Zero-copy form: row u of the query's own tokens, or the pool's row tok; the rows of a pool may span more than 4 GiB.  One path for
    // both: a branch around the loads costs registers and waits at its end (32/8 heads x 64 fp32, 64 tokens over 25k slots 281 / 250 us,
    // 8/2 x 128 fp32 141 / 131; bf16 x 256, 64 tokens over 9.8k slots 218 / 96: 255 registers in memory, 11 without it).
    auto row_off = [&](bool self, bool on, int u, int tok) __attribute__((always_inline)) -> uint64_t {
        unsigned r = (unsigned)(u < n_self ? u : n_self - 1);
        if (!self) r = (unsigned)tok < (unsigned)p.pool_tokens ? (unsigned)tok : (unsigned)p.pool_tokens - 1u;  // never outside the pool
        return on ? (uint64_t)r * (uint64_t)stride : 0;
    };
    // An assembled context, and the query's own tokens, are read through buffers of exactly the split's rows: a lane's offset is its
    // place in the step plus the step's (a scalar), rows past the end read as zero without a trip to memory, and nothing is
    // clamped.  Addresses and clamps as vector arithmetic were 250 of the 700 instructions of a decode step's key step, at 4
    // cycles each and two wavefronts per SIMD.  The loads are cached ones also where no other workgroup reads the rows: an
    // instruction takes half a line of each of 16 keys, the next one the other half (non-temporal: 31 splits of 16k slots
    // 18.2 us, cached 13.5; with every layer's keys cold 18.2 and 16.5).
    const unsigned row_end = (unsigned)(D * E);
    const unsigned ctx_bytes = POOL || nk == 0 ? 0u : (unsigned)((nk - 1) * stride) + row_end;
    const unsigned self_bytes = n_self == 0 ? 0u : (unsigned)((n_self - 1) * stride) + row_end;
    const unsigned k_lane = (unsigned)(l16 * stride) + 16u * (unsigned)kg;         // KR == 4; else 8 bytes per group
    const unsigned v_lane = (unsigned)(4 * kg * stride) + (unsigned)(VW * l16 * E);
    auto load_k = [&](int s, unsigned (&dst)[NK][NJ][KR]) __attribute__((always_inline)) {
        const bool on = s < n_steps, self = s >= n_cs;
        if (POOL) {
#pragma unroll
            for (int b = 0; b < NK; ++b) {
                const char* src = (self ? kself : kctx) + row_off(self, on, SK * (s - n_cs) + 16 * b + l16, tok_k[b]);
#pragma unroll
                for (int j = 0; j < NJ; ++j) {
                    if (KR == 4) {
                        const u32x4 x = *(const u32x4*)(src + 64 * j + 16 * kg);
#pragma unroll
                        for (int i = 0; i < 4; ++i) dst[b][j][i % KR] = x[i];
                    } else {
                        const uint2 x = *(const uint2*)(src + 8 * kg);
                        dst[b][j][0] = x.x;
                        dst[b][j][1 % KR] = x.y;
                    }
                }
            }
            return;
        }
        const buf_rsrc rows_k = make_buffer(self ? kself : kctx, on ? (self ? self_bytes : ctx_bytes) : 0u);
        const unsigned step = (unsigned)(SK * (self ? s - n_cs : s)) * (unsigned)stride;
#pragma unroll
        for (int b = 0; b < NK; ++b) {
            const unsigned at = k_lane + step + (unsigned)(16 * b) * (unsigned)stride;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (KR == 4) {
                    const u32x4 x = buf_load_16(rows_k, at + 64u * j);
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[b][j][i % KR] = x[i];
                } else {
                    const u32x2 x = buf_load_8(rows_k, at - 8u * (unsigned)kg);
                    dst[b][j][0] = x[0];
                    dst[b][j][1 % KR] = x[1];
                }
            }
        }
    };
    // The same through LDS (KL): straight from memory a quarter of a wavefront asks for 16 bytes of 16 rows each, 64 look-ups of
    // cache lines an instruction; row by row it asks for whole lines, 8 of them, and the lanes of the matrix instruction take their chunks
    // from LDS.  A wavefront's keys are its own: no barrier.  (128 KB of K and V rows into every workgroup, 64 / 256 workgroups,
    // out of the last-level cache: 2.8 / 5.0 us with K in the instruction's lanes, 1.65 / 3.9 by rows; out of HBM 3.1 / 6.9 and 2.1 / 7.0.)
    constexpr int KD = KL ? (CM + 1) * RG / RI : 1;  // instructions after which the chunks' places repeat
    unsigned kd_lane[KD];
    if (KL) {
#pragma unroll
        for (int i = 0; i < KD; ++i) {
            const int r = i * RI + lane / CR;
            kd_lane[i] = (unsigned)((lane / CR) * stride) + 16u * (unsigned)((lane % CR) ^ ((r / RG) & CM));
        }
    }
    auto dma_k = [&](int s, char* buf) __attribute__((always_inline)) {
        const bool on = s < n_steps, self = s >= n_cs;
        const buf_rsrc rows_k = make_buffer(self ? kself : kctx, on ? (self ? self_bytes : ctx_bytes) : 0u);
        const unsigned step = (unsigned)(SK * (self ? s - n_cs : s)) * (unsigned)stride;
#pragma unroll
        for (int i = 0; i < (KL ? KS_BYTES / 1024 : 0); ++i)
            buf_load_lds_16(rows_k, buf + i * 1024, kd_lane[i % KD] + step + (unsigned)(i * RI) * (unsigned)stride);
    };
    auto take_k = [&](const char* buf, unsigned (&dst)[NK][NJ][KR]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < NK; ++b)
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const int r = 16 * b + l16;
                const u32x4 x = *(const u32x4*)(buf + r * RB + (((4 * j + kg) ^ ((r / RG) & CM)) << 4));
#pragma unroll
                for (int i = 0; i < 4; ++i) dst[b][j][i % KR] = x[i];
            }
    };
    auto load_v = [&](int s, unsigned (&dst)[NV][DG][VR]) __attribute__((always_inline)) {
        const bool on = s < n_steps, self = s >= n_cs;
        if (POOL) {
#pragma unroll
            for (int r = 0; r < NV; ++r) {
                const char* src = (self ? vself : vctx) + row_off(self, on, SK * (s - n_cs) + 16 * (r >> 2) + 4 * kg + (r & 3), tok_v[r]);
#pragma unroll
                for (int dg = 0; dg < DG; ++dg) {
                    const char* q = src + (16 * VW * dg + VW * l16) * E;
                    if (VR == 4) {
                        const u32x4 x = *(const u32x4*)q;
#pragma unroll
                        for (int i = 0; i < 4; ++i) dst[r][dg][i % VR] = x[i];
                    } else if (VR == 2) {
                        const uint2 x = *(const uint2*)q;
                        dst[r][dg][0] = x.x;
                        dst[r][dg][1 % VR] = x.y;
                    } else if (VW * E == 4) {
                        dst[r][dg][0] = D == 8 && l16 >= 8 ? 0u : *(const unsigned*)(D == 8 && l16 >= 8 ? src : q);
                    } else {
                        dst[r][dg][0] = (unsigned)*(const unsigned short*)q << 16;  // bf16, one column
                    }
                }
            }
            return;
        }
        const buf_rsrc rows_v = make_buffer(self ? vself : vctx, on ? (self ? self_bytes : ctx_bytes) : 0u);
        const unsigned step = (unsigned)(SK * (self ? s - n_cs : s)) * (unsigned)stride;
#pragma unroll
        for (int r = 0; r < NV; ++r) {
            const unsigned at = v_lane + step + (unsigned)(16 * (r >> 2) + (r & 3)) * (unsigned)stride;
#pragma unroll
            for (int dg = 0; dg < DG; ++dg) {
                const unsigned q = at + (unsigned)(16 * VW * dg * E);
                if (VR == 4) {
                    const u32x4 x = buf_load_16(rows_v, q);
#pragma unroll
                    for (int i = 0; i < 4; ++i) dst[r][dg][i % VR] = x[i];
                } else if (VR == 2) {
                    const u32x2 x = buf_load_8(rows_v, q);
                    dst[r][dg][0] = x[0];
                    dst[r][dg][1 % VR] = x[1];
                } else if (VW * E == 4) {
                    const unsigned x = buf_load_4(rows_v, q);
                    dst[r][dg][0] = D == 8 && l16 >= 8 ? 0u : x;
                } else {
                    dst[r][dg][0] = (unsigned)buf_load_2(rows_v, q) << 16;  // bf16, one column
                }
            }
        }
    };
    // bf16: column c of two V rows in one register, the first in the low half
    auto v_pair = [&](const unsigned (&x)[VR], const unsigned (&y)[VR], int c) __attribute__((always_inline)) -> unsigned {
        const unsigned a = x[(c >> 1) % VR], b = y[(c >> 1) % VR];
        return __builtin_amdgcn_perm(b, a, (c & 1) || VW == 1 ? 0x07060302u : 0x05040100u);
    };

    // ---- rotation of a lane's pieces of a key to position a (Eq. rope_encoding); bf16 results rounded to
    // nearest even, as a cache would hold them.  The partner of column d is d +- D/2: piece j +- NJ/2 of the same lane, or,
    // where a row is a single piece per lane, the lane two groups on.
    auto get = [&](const unsigned (&w)[KR], int c) __attribute__((always_inline)) -> float {
        if (!BF) return __uint_as_float(w[c % KR]);
        return (c & 1) ? __uint_as_float(w[(c >> 1) % KR] & 0xffff0000u) : __uint_as_float(w[(c >> 1) % KR] << 16);
    };
    auto put2 = [&](unsigned (&w)[KR], int c, float a, float b) __attribute__((always_inline)) {
        if (BF) {
            w[(c >> 1) % KR] = pack2_bf16(a, b);
        } else {
            w[c % KR] = __float_as_uint(a);
            w[(c + 1) % KR] = __float_as_uint(b);
        }
    };
    auto rotate = [&](unsigned (&x)[NJ][KR], int64_t a) __attribute__((always_inline)) {
        const float2* th = p.tab_hi + (a >> kRopeLoBits) * (D / 2);
        const float2* tl = p.tab_lo + (a & (kRopeLo - 1)) * (D / 2);
        constexpr int NP = NJ > 1 ? NJ / 2 : 1;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int f0 = NJ > 1 ? 4 * KW * j + KW * kg : KW * (kg & 1);
#pragma unroll
            for (int c = 0; c < KW; c += 2) {
                const f32x4 h = *(const f32x4*)(th + f0 + c), l = *(const f32x4*)(tl + f0 + c);
                const float c0 = h[0] * l[0] - h[1] * l[1], s0 = h[1] * l[0] + h[0] * l[1];
                const float c1 = h[2] * l[2] - h[3] * l[3], s1 = h[3] * l[2] + h[2] * l[3];
                if (NJ > 1) {
                    const float a0 = get(x[j], c), a1 = get(x[j], c + 1);
                    const float b0 = get(x[(j + NP) % NJ], c), b1 = get(x[(j + NP) % NJ], c + 1);
                    put2(x[j], c, a0 * c0 - b0 * s0, a1 * c1 - b1 * s1);
                    put2(x[(j + NP) % NJ], c, b0 * c0 + a0 * s0, b1 * c1 + a1 * s1);
                } else {
                    const float a0 = get(x[0], c), a1 = get(x[0], c + 1);
                    const float b0 = __shfl_xor(a0, 32, 64), b1 = __shfl_xor(a1, 32, 64);
                    const float t0 = kg < 2 ? -s0 : s0, t1 = kg < 2 ? -s1 : s1;
                    put2(x[0], c, a0 * c0 + b0 * t0, a1 * c1 + b1 * t1);
                }
            }
        }
    };

    // ---- query rows: rotated once per workgroup (a thread per pair of 16-byte chunks, halves of a head apart), through LDS into the
    // fragments of every wavefront; the first steps' keys and values are requested behind them
    constexpr int CH = D * E / 32, NCH = 2 * CH;  // 16-byte chunks of half a head, of a head
    constexpr int QI = (TR * CH + T - 1) / T;
    auto q_chunk = [&](int row, int c) __attribute__((always_inline)) -> char* { return qs + (row * NCH + (c ^ (row & (NCH - 1)))) * 16; };
    u32x4 qa[QI], qb[QI];
    f32x4 th[QI][KP / 2], tl[QI][KP / 2];
#pragma unroll
    for (int i = 0; i < QI; ++i) {
        if (wave * 64 + i * T >= TR * CH) break;
        const int r = (tid + i * T) / CH < TR ? (tid + i * T) / CH : TR - 1, c = tid % CH;
        const int rc = row0 + r < rows ? row0 + r : rows - 1;
        const int j = p.div_g.of(rc);
        const char* src = it.q + (((int64_t)j * p.n_q_heads + hk * g + (rc - j * g)) * D) * E + 16 * c;
        qa[i] = *(const u32x4*)src;
        qb[i] = *(const u32x4*)(src + 16 * CH);
        const int64_t a = (int64_t)it.q_pos0 + j;
        const f32x4* h4 = (const f32x4*)(p.tab_hi + (a >> kRopeLoBits) * (D / 2) + KP * c);
        const f32x4* l4 = (const f32x4*)(p.tab_lo + (a & (kRopeLo - 1)) * (D / 2) + KP * c);
#pragma unroll
        for (int e = 0; e < KP / 2; ++e) {
            th[i][e] = h4[e];
            tl[i][e] = l4[e];
        }
    }
    unsigned kf[KL ? 1 : NB][NK][NJ][KR];
    char* const kw0 = ks0 + (KL ? wave * OS_BYTES : 0);
    char* const kw1 = ks1 + (KL ? wave * KS_BYTES : 0);
    // keys of step s into buffer b; LDS: every read of what the buffer held has returned
    auto get_k = [&](int s, int b) __attribute__((always_inline)) {
        if (!KL) {
            load_k(s, kf[b % (KL ? 1 : NB)]);
            return;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        dma_k(s, b == 0 ? kw0 : kw1);
    };
    unsigned vf[NBV][NV][DG][VR];
    fetch_tok(wave);
    take_tok();
    if (TOK2) fetch_tok(wave + W);
    get_k(wave, 0);
    if (NBV > 1 && !KL) {
        load_v(wave, vf[0]);
        if (!TOK2) fetch_tok(wave + W);
        take_tok();
    }
#pragma unroll
    for (int i = 0; i < QI; ++i) {
        if (wave * 64 + i * T >= TR * CH) break;
#pragma unroll
        for (int e = 0; e < KP / 2; ++e) {  // frequencies 2e and 2e + 1 of the chunk
            const f32x4 h = th[i][e], l = tl[i][e];
            const float c0 = h[0] * l[0] - h[1] * l[1], s0 = h[1] * l[0] + h[0] * l[1];
            const float c1 = h[2] * l[2] - h[3] * l[3], s1 = h[3] * l[2] + h[2] * l[3];
            if (BF) {
                const float a0 = __uint_as_float(qa[i][e] << 16), a1 = __uint_as_float(qa[i][e] & 0xffff0000u);
                const float b0 = __uint_as_float(qb[i][e] << 16), b1 = __uint_as_float(qb[i][e] & 0xffff0000u);
                qa[i][e] = pack2_bf16((a0 * c0 - b0 * s0) * p.q_scale, (a1 * c1 - b1 * s1) * p.q_scale);
                qb[i][e] = pack2_bf16((b0 * c0 + a0 * s0) * p.q_scale, (b1 * c1 + a1 * s1) * p.q_scale);
            } else {
                const float a0 = __uint_as_float(qa[i][2 * e % 4]), a1 = __uint_as_float(qa[i][(2 * e + 1) % 4]);
                const float b0 = __uint_as_float(qb[i][2 * e % 4]), b1 = __uint_as_float(qb[i][(2 * e + 1) % 4]);
                qa[i][2 * e % 4] = __float_as_uint((a0 * c0 - b0 * s0) * p.q_scale);
                qa[i][(2 * e + 1) % 4] = __float_as_uint((a1 * c1 - b1 * s1) * p.q_scale);
                qb[i][2 * e % 4] = __float_as_uint((b0 * c0 + a0 * s0) * p.q_scale);
                qb[i][(2 * e + 1) % 4] = __float_as_uint((b1 * c1 + a1 * s1) * p.q_scale);
            }
        }
        if (tid + i * T < TR * CH) {
            const int r = (tid + i * T) / CH, c = tid % CH;
            *(u32x4*)q_chunk(r, c) = qa[i];
            *(u32x4*)q_chunk(r, c + CH) = qb[i];
        }
    }
    // (a barrier that leaves the loads of keys and values in flight)
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    // (V behind the barrier: the wavefronts that take the query rows stand in line with the others' requests, and 64 KB of keys are
    // enough to be in flight until then: 1357 calls, V before the barrier 2 % faster than without LDS, behind it 4 %)
    if (NBV > 1 && KL) load_v(wave, vf[0]);
    unsigned qf[NR][NJ][KR];
    int jrow[NR];
#pragma unroll
    for (int nr = 0; nr < NR; ++nr) {
        const int row = row0 + 16 * nr + l16;
        jrow[nr] = p.div_g.of(row < rows ? row : rows - 1);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            if (KR == 4) {
                const u32x4 x = *(const u32x4*)q_chunk(16 * nr + l16, 4 * jj + kg);
#pragma unroll
                for (int i = 0; i < 4; ++i) qf[nr][jj][i % KR] = x[i];
            } else {
                const u32x2 x = *(const u32x2*)(q_chunk(16 * nr + l16, kg >> 1) + 8 * (kg & 1));
                qf[nr][jj][0] = x[0];
                qf[nr][jj][1 % KR] = x[1];
            }
        }
    }

    f32x4 o[NR][DB];
    float m_run[NR], l_run[NR];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int nr = 0; nr < NR; ++nr) {
            m_run[nr] = -INFINITY;
            l_run[nr] = 0.f;
#pragma unroll
            for (int b = 0; b < DB; ++b) o[nr][b] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    clear();

    // keys that come un-rotated, turned to their positions; loads return in order, and behind the next step's rows the tables' entries
    // are waited for with them; all: blocks that no row sees as well
    auto turn = [&](int s, unsigned (&k)[NK][NJ][KR], bool all = false) __attribute__((always_inline)) {
        const bool self = s >= n_cs;
#pragma unroll
        for (int kb = 0; kb < NK; ++kb) {
            // Blocks past the own tokens are masked, whatever they hold, and not turned, but for the gathered forms that are slower with the
            // branch: fp32, and bf16 from 64 columns on, which do best with one rotation of either kind of keys.  With / without it,
            // us: fp32 x 128, 32/8 heads, 100 tokens over 7.9k slots 336 / 280, 8/2 heads, 64 over 7.9k 52.0 / 43.8, 24 over 154 11.8 / 10.9;
            // fp32 x 64, 4/2 heads, 24 over 154 7.7 / 6.9; bf16 x 64, 24 over 260 8.7 / 8.0.  (bf16 x 16 and x 32 with one rotation: registers for
            // half the workgroups, 256 tokens of 32/8 heads over 24k 270 -> 301 and 552 -> 569.)
            const bool seen = SK * (s - n_cs) + 16 * kb < n_self;
            if (POOL && BF && D >= 64) {
                rotate(k[kb], (self ? (int64_t)it.q_pos0 + SK * (s - n_cs) : p.ctx_pos0 + k0 + SK * s) + 16 * kb + l16);
            } else if (self) {
                if ((POOL && !BF) || all || seen) rotate(k[kb], (int64_t)it.q_pos0 + SK * (s - n_cs) + 16 * kb + l16);
            } else if (POOL) {
                rotate(k[kb], p.ctx_pos0 + k0 + SK * s + 16 * kb + l16);
            }
        }
    };

    // key_by_key: the second product without matrix instructions (for values that are not finite, see below)
    auto compute = [&](int s, unsigned (&k)[NK][NJ][KR], unsigned (&v)[NV][DG][VR], auto key_by_key) __attribute__((always_inline)) {
        const bool self = s >= n_cs;  // wavefront-uniform
        f32x4 sc[NK][NR];
#pragma unroll
        for (int kb = 0; kb < NK; ++kb) {
#pragma unroll
            for (int nr = 0; nr < NR; ++nr) sc[kb][nr] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if (BF && KR == 4) {
                    const u32x4 a = {k[kb][j][0], k[kb][j][1 % KR], k[kb][j][2 % KR], k[kb][j][3 % KR]};
#pragma unroll
                    for (int nr = 0; nr < NR; ++nr) {
                        const u32x4 b = {qf[nr][j][0], qf[nr][j][1 % KR], qf[nr][j][2 % KR], qf[nr][j][3 % KR]};
                        sc[kb][nr] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                                             __builtin_bit_cast(bf16x8, b), sc[kb][nr], 0, 0, 0);
                    }
                } else if (BF) {
                    const uint2 a = {k[kb][j][0], k[kb][j][1 % KR]};
#pragma unroll
                    for (int nr = 0; nr < NR; ++nr) {
                        const uint2 b = {qf[nr][j][0], qf[nr][j][1 % KR]};
                        sc[kb][nr] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a),
                                                                               __builtin_bit_cast(s16x4, b), sc[kb][nr], 0, 0, 0);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < KR; ++i)
#pragma unroll
                        for (int nr = 0; nr < NR; ++nr)
                            sc[kb][nr] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(k[kb][j][i]), __uint_as_float(qf[nr][j][i]),
                                                                              sc[kb][nr], 0, 0, 0);
                }
            }
        }
        const int u = SK * (self ? s - n_cs : s) + 4 * kg;
#pragma unroll
        for (int nr = 0; nr < NR; ++nr) {
            if (self || SK * s + SK > nk) {
                const int lim = self ? jrow[nr] + 1 : nk;
#pragma unroll
                for (int kb = 0; kb < NK; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (u + 16 * kb + r >= lim) sc[kb][nr][r] = -INFINITY;
            }
            float mx = fmaxf(fmaxf(sc[0][nr][0], sc[0][nr][1]), fmaxf(sc[0][nr][2], sc[0][nr][3]));
            if (NK == 2)
                mx = fmaxf(mx, fmaxf(fmaxf(sc[NK - 1][nr][0], sc[NK - 1][nr][1]), fmaxf(sc[NK - 1][nr][2], sc[NK - 1][nr][3])));
            // the reference maximum of a row follows lazily: it moves when a score exceeds it by more than 2^8
            if (__builtin_amdgcn_ballot_w64(mx > m_run[nr] + 8.0f)) {
                mx = max_xhalf(max_xrow(mx));
                const float m_new = fmaxf(m_run[nr], mx);
                const float alpha = m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_run[nr] - m_new);
                m_run[nr] = m_new;
                l_run[nr] *= alpha;
#pragma unroll
                for (int b = 0; b < DB; ++b)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[nr][b][r] *= alpha;
            }
            const float m_use = m_run[nr] == -INFINITY ? 0.f : m_run[nr];
#pragma unroll
            for (int kb = 0; kb < NK; ++kb) {
#pragma unroll
                for (int r = 0; r < 4; ++r) sc[kb][nr][r] = __builtin_amdgcn_exp2f(sc[kb][nr][r] - m_use);
                l_run[nr] += (sc[kb][nr][0] + sc[kb][nr][1]) + (sc[kb][nr][2] + sc[kb][nr][3]);
            }
        }
        if constexpr (decltype(key_by_key)::value) {
#pragma unroll 1
            for (int kq = 0; kq < 4; ++kq)
#pragma unroll
                for (int kr = 0; kr < NV; ++kr) {  // key 16 * (kr / 4) + 4 * kq + kr % 4 of the step
                    const int key = SK * (self ? s - n_cs : s) + 16 * (kr >> 2) + 4 * kq + (kr & 3);
                    float w[NR];
#pragma unroll
                    for (int nr = 0; nr < NR; ++nr) w[nr] = __shfl(sc[kr >> 2][nr][kr & 3], 16 * kq + l16, 64);
#pragma unroll
                    for (int dg = 0; dg < DG; ++dg)
#pragma unroll
                        for (int i = 0; i < 4; ++i)  // a lane's columns 16 * VW * dg + VW * (4 * kg + i) + c
#pragma unroll
                            for (int x = 0; x < VR; ++x) {
                                const unsigned y = __shfl(v[kr][dg][x], 16 * kq + 4 * kg + i, 64);
                                constexpr int CX = BF && VW > 1 ? 2 : 1;  // columns of a register
#pragma unroll
                                for (int c = 0; c < CX; ++c) {
                                    const float val = __uint_as_float(CX == 1 ? y : c == 0 ? y << 16 : y & 0xffff0000u);
#pragma unroll
                                    for (int nr = 0; nr < NR; ++nr) {
                                        f32x4& acc = o[nr][dg * VW + CX * x + c];
                                        acc[i] = key < (self ? jrow[nr] + 1 : nk) ? fmaf(w[nr], val, acc[i]) : acc[i];
                                    }
                                }
                            }
                }
        } else if constexpr (BF) {
            // pb[nr][i]: piece i of the weights, slot 4*kb + r of a lane = key 16*kb + 4*kg + r, as V has them
            unsigned pb[NR][NP][2 * NK];
#pragma unroll
            for (int nr = 0; nr < NR; ++nr)
#pragma unroll
                for (int w = 0; w < 2 * NK; ++w) {
                    float x = sc[w >> 1][nr][2 * (w & 1)], y = sc[w >> 1][nr][2 * (w & 1) + 1];
#pragma unroll
                    for (int i = 0; i < NP; ++i) {
                        if (NP == 2 && i == 1) {  // rounded: 2^-17 of the weight
                            pb[nr][i][w] = pack2_bf16(x, y);
                            continue;
                        }
                        // the upper 8 of the bits that are left, exactly
                        pb[nr][i][w] = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);
                        x -= __uint_as_float(__float_as_uint(x) & 0xffff0000u);
                        y -= __uint_as_float(__float_as_uint(y) & 0xffff0000u);
                    }
                }
#pragma unroll
            for (int dg = 0; dg < DG; ++dg)
#pragma unroll
                for (int c = 0; c < VW; ++c) {
                    unsigned a[2 * NK];
#pragma unroll
                    for (int w = 0; w < 2 * NK; ++w) a[w] = v_pair(v[2 * w][dg], v[2 * w + 1][dg], c);
#pragma unroll
                    for (int i = 0; i < NP; ++i)
#pragma unroll
                        for (int nr = 0; nr < NR; ++nr) {
                            f32x4& acc = o[nr][dg * VW + c];
                            if (NK == 2) {
                                const u32x4 av = {a[0], a[1], a[2 % (2 * NK)], a[3 % (2 * NK)]};
                                const u32x4 bv = {pb[nr][i][0], pb[nr][i][1], pb[nr][i][2 % (2 * NK)], pb[nr][i][3 % (2 * NK)]};
                                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, av), __builtin_bit_cast(bf16x8, bv),
                                                                              acc, 0, 0, 0);
                            } else {
                                const uint2 av = {a[0], a[1]}, bv = {pb[nr][i][0], pb[nr][i][1]};
                                acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, av), __builtin_bit_cast(s16x4, bv),
                                                                                acc, 0, 0, 0);
                            }
                        }
                }
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int dg = 0; dg < DG; ++dg)
#pragma unroll
                    for (int c = 0; c < VW; ++c) {
                        const float a = __uint_as_float(v[r][dg][c % VR]);
#pragma unroll
                        for (int nr = 0; nr < NR; ++nr)
                            o[nr][dg * VW + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sc[0][nr][r], o[nr][dg * VW + c], 0, 0, 0);
                    }
        }
    };

    if (wave < n_steps) {  // (said once for both loops: what only they need is then computed under it)
        // Steps in pairs, one buffer each, and the odd one behind the loop: a loop that could be left between the two has the
        // compiler wait at its head for loads that only that way out leaves behind, and a wavefront with one step loads no
        // second one (one step per wavefront: 7.2 -> 6.6 us of a call, 10.3 -> 9.6).
        int s = wave;
        // (bf16 x 32 turns blocks that no row sees, but for the step behind the loop: 32/8 heads, 94 tokens over 6.4k slots 28.1 -> 27.3 us, 111 over 7.2k
        // 31.2 -> 30.6, before any block was left out 27.6 and 30.8; small calls lose 1 to 2 % of the 10 that this gave them.)
        constexpr bool kLoopTurnsAll = BF && D == 32 && !POOL;
        auto step = [&](int b) __attribute__((always_inline)) {
            const int kb = KL ? 0 : b;
            if (!LATE && !KL) turn(s, kf[kb], kLoopTurnsAll);
            if (NBV == 1) {
                load_v(s, vf[0]);
                fetch_tok(s + W);
                take_tok();
            }
            if (TOK2) fetch_tok(s + 2 * W);
            get_k(s + W, 1 - b);
            if (NBV > 1) {
                load_v(s + W, vf[(1 - b) % NBV]);
                if (!TOK2) fetch_tok(s + 2 * W);
                take_tok();
            }
            if (KL) {
                __builtin_amdgcn_sched_barrier(0);  // the next step's loads first
                take_k(b == 0 ? kw0 : kw1, kf[0]);
            }
            if (LATE || KL) turn(s, kf[kb], kLoopTurnsAll);
            compute(s, kf[kb], vf[b % NBV], std::false_type{});
            s += W;
        };
        while (s + W < n_steps) {
            step(0);
            step(1);
        }
        if (s < n_steps) {
            if (KL) take_k(kw0, kf[0]);
            turn(s, kf[0]);
            if (NBV == 1) load_v(s, vf[0]);
            compute(s, kf[0], vf[0], std::false_type{});
        }

        // A matrix product multiplies every V row of its step with every query row: a V that is not finite makes NaN of the
        // rows that must not see its token (weight 0) and, where P is in pieces, an infinite one of those whose weight
        // leaves a piece 0 (a weight of 1 leaves two).  A wavefront whose sums hold a NaN therefore takes its keys a second
        // time, one by one, each only for the rows that see it.  Looking for NaN costs a call without any 0.1 to 0.2 us
        // (kernel alone: 64 query tokens of 32/8 heads x 64 over 6.6k slots 22.2 -> 22.5 us; head dimension 256, where the
        // second loop's registers spill, up to 0.6 us of 11 to 19).
        bool nan = false;
#pragma unroll
        for (int nr = 0; nr < NR; ++nr)
#pragma unroll
            for (int b = 0; b < DB; ++b)
                nan |= __builtin_isunordered(o[nr][b][0], o[nr][b][1]) || __builtin_isunordered(o[nr][b][2], o[nr][b][3]);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(nan) != 0, 0)) {
            clear();
#pragma unroll 1
            for (int s = wave; s < n_steps; s += W) {
                fetch_tok(s);
                take_tok();
                get_k(s, 0);
                load_v(s, vf[0]);
                if (KL) take_k(kw0, kf[0]);
                turn(s, kf[0]);
                compute(s, kf[0], vf[0], std::true_type{});
            }
        }
    }

    // ---- the wavefronts' states meet
#pragma unroll
    for (int nr = 0; nr < NR; ++nr) {
        float l = l_run[nr];
        l = sum_xhalf(sum_xrow(l));
        if (kg == 0) wml[wave][16 * nr + l16] = make_float2(m_run[nr], l);
#pragma unroll
        for (int s = 0; s < DB; ++s) {
            f32x4 x;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int f = 4 * (s % VW) + i;  // index in the lane's run of 4 * VW columns: column VW * r + c
                x[i] = o[nr][(s / VW) * VW + f % VW][f / VW];
            }
            os[wave][nr * DB + s][lane] = x;
        }
    }
    __syncthreads();
    float wgt[NR][W], m_wg[NR], l_wg[NR];
#pragma unroll
    for (int nr = 0; nr < NR; ++nr) {
        float2 ml[W];
#pragma unroll
        for (int w = 0; w < W; ++w) ml[w] = wml[w][16 * nr + l16];
        float M = ml[0].x;
#pragma unroll
        for (int w = 1; w < W; ++w) M = fmaxf(M, ml[w].x);
        float L = 0.f;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            wgt[nr][w] = ml[w].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - M);
            L += wgt[nr][w] * ml[w].y;
        }
        m_wg[nr] = M;
        l_wg[nr] = L;
    }
    const int64_t unit = it.unit0 + (int64_t)rt * hkv + hk;
    // partials of the unit, [split][row][column]: at most 64 splits of 32 rows of 256 columns
    const buf_rsrc parts = make_buffer(p.part_o + unit * p.max_split * (TR * D), (unsigned)(n_split * (TR * D) * 4));
    auto store_out = [&](int row, int d0, f32x4 y) __attribute__((always_inline)) {
        const int j = p.div_g.of(row);
        const int64_t e = ((int64_t)j * p.n_q_heads + hk * g + (row - j * g)) * D + d0;
        if (BF) *(uint2*)(it.out + e * 2) = make_uint2(pack2_bf16(y[0], y[1]), pack2_bf16(y[2], y[3]));
        else *(f32x4*)(it.out + e * 4) = y;
    };
    for (int s = wave; s < NS; s += W) {
        const int nr = s / DB, sl = s % DB;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float Lr = 1.f;
#pragma unroll
        for (int n2 = 0; n2 < NR; ++n2)
            if (n2 == nr) {
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    const f32x4 x = os[w][s][lane];
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[i] += wgt[n2][w] * x[i];
                }
                Lr = l_wg[n2];
            }
        const int row = row0 + 16 * nr + l16;
        const int d0 = 16 * VW * (sl / VW) + 4 * VW * kg + 4 * (sl % VW);
        if (row < rows && d0 < D) {
            if (n_split == 1) {
                const float inv = 1.0f / Lr;
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] *= inv;
                store_out(row, d0, acc);
            } else {
                buf_store_16<kCacheDevice>(parts, (unsigned)((split * TR + row - row0) * D + d0) * 4u, __builtin_bit_cast(u32x4, acc));
            }
        }
    }
    if (n_split == 1) return;

    // ---- merge over the splits, by the workgroup that arrives last at the unit's counter.  Nobody waits: a workgroup that
    // waited for the others, to merge a share of the rows, would hold its compute unit while workgroups of other streams' launches
    // -- or of its own -- need it.  (Waits of up to 10 us, nobody / all wait: one token over 16k slots of 28/4 heads 15.6 / 13.8 us
    // alone, but 13.1 / 13.8, 10.0 / 21.1 and 9.0 / 21.1 us a call on 2, 3 and 4 streams.)
    float* const pml = p.part_ml + unit * p.max_split * (TR * 2);
    if (wave == 0 && kg == 0) {
#pragma unroll
        for (int nr = 0; nr < NR; ++nr) stream_store2(pml + (split * TR + 16 * nr + l16) * 2, m_wg[nr], l_wg[nr]);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wavefront's partials have reached memory
    __syncthreads();
    if (tid == 0) {
        unsigned* const word = p.counters + unit * p.counter_stride;
        const unsigned before = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        last_flag = before == (unsigned)n_split - 1u ? 1 : 0;
        if (last_flag) __hip_atomic_store(word, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last_flag) return;

    // Without branches over absent splits: a taken branch to code that no wavefront of the compute unit has run yet is 70 ns, loads past
    // the end of a buffer and weights of 0 are none.  Calls over cold contexts, with such branches / without, us: 28/4 heads, one token over 16k
    // slots 15.1 / 13.4, 32/8 heads over 4k 9.8 / 8.8, 24 tokens over 830 9.7 / 8.5, fp32 x 128, 32 tokens over 2k 13.8 / 11.7.  (More splits in
    // flight made it longer, not shorter: 16 or 24 of them, with branches, 1.5 and 12 % of such calls.)
    const int n_rows = rows - row0 < TR ? rows - row0 : TR;
    const int e4 = n_rows * (D / 4);  // 16-byte pieces of the output rows
    constexpr int PB = 8;             // splits in flight per thread, twice
    // Threads in groups of a power of two, one for every piece of a pass; the groups take the splits between them, up to 8 splits one group.  No
    // round of loads behind the last one, and that one's sum outside the loop.  With eight groups and a round more whatever there is / now, us: 4/2
    // fp32 heads x 64, 32 queries of one token over 250 to 500 slots, 4 splits 8.5 / 7.9 (before the merge lost its branches 8.2); 8/2 x 128, 32
    // tokens over 2.5k, 16 splits 11.8 / 11.4, 28/4 heads, one over 20k, 32 splits 11.8 / 11.6 (the round behind a branch in the loop: 12.2, 12.3).
    const int lg_t = 31 - __builtin_clz(T), lg_e = e4 > 1 ? 32 - __builtin_clz(e4 - 1) : 0;
    const int lg_g = n_split > PB ? 32 - __builtin_clz((n_split - 1) / PB) : 0;
    const int lg_pe = lg_e < lg_t - lg_g ? lg_t - lg_g : lg_e < lg_t ? lg_e : lg_t;
    const int pe = 1 << lg_pe, ng = T >> lg_pe;  // pieces of a pass; at most 8 groups
    const int grp = tid >> lg_pe, ei = tid & (pe - 1);
    const unsigned split_bytes = TR * D * 4;
    auto pieces = [&](int e, int s0, f32x4 (&x)[PB]) __attribute__((always_inline)) {
        const unsigned at = e < e4 ? (unsigned)(s0 + grp) * split_bytes + 16u * (unsigned)e : 0xf0000000u;
#pragma unroll
        for (int b = 0; b < PB; ++b) x[b] = __builtin_bit_cast(f32x4, buf_load_16<kCacheDevice>(parts, at + (unsigned)(b * ng) * split_bytes));
    };
    // weights of the splits, a wavefront per row and a lane per split: sw[s][row] = 2^(m_s - M) / L, 0 for absent splits
    const buf_rsrc mls = make_buffer(pml, (unsigned)(n_split * (TR * 8)));
    constexpr int WR = (TR + W - 1) / W;  // rows of a wavefront
    u32x2 ml[WR];
#pragma unroll
    for (int i = 0; i < WR; ++i) ml[i] = buf_load_8<kCacheDevice>(mls, (unsigned)((lane * TR + wave + i * W) * 8));
    f32x4 x[PB];
    pieces(ei, 0, x);  // requested with the (m, l)
#pragma unroll
    for (int i = 0; i < WR; ++i) {
        const float m = lane < n_split ? __uint_as_float(ml[i][0]) : -INFINITY;
        const float M = wave_max(m);
        const float w = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - M);
        const float L = wave_sum(w == 0.f ? 0.f : w * __uint_as_float(ml[i][1]));
        sw[lane][wave + i * W] = w == 0.f ? 0.f : w * (1.0f / L);
    }
    __syncthreads();
    f32x4* const red = (f32x4*)ks0;  // a piece per thread
    for (int e0 = 0; e0 < e4; e0 += pe) {
        const int e = e0 + ei;
        const int row = e / (D / 4);
        if (e0 != 0) pieces(e, 0, x);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        auto add = [&](int s0) __attribute__((always_inline)) {  // (s0 + grp + b * ng < 64: PB * ng divides it)
            const float* wr = &sw[s0 + grp][row < TR ? row : 0];
#pragma unroll
            for (int b = 0; b < PB; ++b) {
                const float w = wr[b * ng * TR];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] += w * x[b][i];
            }
        };
        int s0 = 0;
        for (; s0 + PB * ng < n_split; s0 += PB * ng) {
            f32x4 y[PB];
            pieces(e, s0 + PB * ng, y);
            add(s0);
#pragma unroll
            for (int b = 0; b < PB; ++b) x[b] = y[b];
        }
        add(s0);
        if (ng > 1) {  // (then this is the only pass)
            red[tid] = acc;
            __syncthreads();
            if (grp != 0) continue;
            for (int k = 1; k < ng; ++k) {
                const f32x4 z = red[tid + (k << lg_pe)];
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[i] += z[i];
            }
        }
        if (e < e4) store_out(row0 + row, 4 * (e - row * (D / 4)), acc);
    }
}

template <int DTYPE, int D, int NR>
static hipError_t launch_stream_form(const StreamLaunch& s, hipStream_t stream) {
    auto fill = [&](auto& a) {
        a.tab_lo = s.tab_lo;
        a.tab_hi = s.tab_hi;
        a.part_o = s.part_o;
        a.part_ml = s.part_ml;
        a.counters = s.counters;
        a.slot_src = s.slot_src;
        a.ctx_pos0 = s.ctx_pos0;
        a.n_q_heads = s.n_q_heads;
        a.n_kv_heads = s.n_kv_heads;
        a.g = s.n_q_heads / s.n_kv_heads;
        a.div_hkv = fast_div(s.n_kv_heads);
        a.div_g = fast_div(a.g);
        a.max_split = s.max_split;
        a.counter_stride = s.counter_stride;
        a.pool_tokens = s.pool_tokens;
        a.q_scale = s.q_scale;
        for (int i = 0; i < s.n_items; ++i) a.it[i] = s.items[i];
        for (int i = s.n_items; i < (int)(sizeof(a.it) / sizeof(a.it[0])); ++i) a.it[i].block0 = INT32_MAX;  // (nobody's)
    };
    const dim3 grid((unsigned)s.n_wgs), block(kStreamWaves * 64);
    if (s.n_items == 1) {
        StreamArgs<1> a;
        fill(a);
        if (s.slot_src) {
            if constexpr (DTYPE == ADAPSHOT_BF16 && D == 128) return hipErrorInvalidValue;  // the tile kernel's zero-copy form
            else launch_kernel((attn_stream_kernel<DTYPE, D, NR, true, 1>), grid, block, stream, a);
        } else launch_kernel((attn_stream_kernel<DTYPE, D, NR, false, 1>), grid, block, stream, a);
    } else {
        if (s.slot_src) return hipErrorInvalidValue;
        StreamArgs<kStreamItems> a;
        fill(a);
        launch_kernel((attn_stream_kernel<DTYPE, D, NR, false, kStreamItems>), grid, block, stream, a);
    }
    return hipGetLastError();
}

}  // namespace adapshot
