// The pass of relevance ranking over the keys of the whole pool (bf16, head_dim 128; Eq. attention_score): for every
// query row and every segment (what one split of the pool holds of one shot) the sum of 2^(s - m) over the segment's
// keys, and per split the row's reference maximum m and sum.  rank_weights and rank_reduce turn them into scores.
//
// Workgroup = (kv head, tile of 256 * NR rows, split of the pool's keys); 8 wavefronts, two per SIMD, each owning 32 * NR
// rows for the whole key loop.  S^T = K . Q^T as in the attention kernel (a query row lives in a lane column, A = K from
// LDS, B = Q in registers), and that is the only product: there are no values.  A block of 32 keys leaves a lane 16 scores
// of its row, their exponentials are added in fp32 to the running sum of the segment, and a segment that ends inside the
// block is cut out with 0 / 1 factors that depend on the key alone.  When a segment ends its sum leaves: lanes l and l^32
// add their halves (two row blocks with one swap) and a store instruction writes 32 * NR consecutive rows.
//
// No maximum is taken in the key loop.  fp32 sums do not care how large the exponentials are until they overflow, so the
// reference of a row is 0 when its first block's maximum lies within 2^+-40 (the usual case: the exponentials then need no
// subtraction either), else that maximum, and a block is only looked at again when a sum leaves 2^80: its scores are
// computed a second time from the tile still in LDS, the reference of the rows that exceed theirs moves, and what has left
// for this split already is scaled in place.
//
// The exponentials of a block are interleaved with the products of the next one, two behind every matrix instruction, in one
// straight run of instructions: left to two wavefronts of a SIMD in opposite phases they hardly overlapped (matrix cores
// and vector ALU busy together 14 % of the time, now 29 %), and every branch in the run costs more than what it saves.
// A tile stays in LDS for one tile longer than its products need it, for the second look.
//
// What bounds it: matrix cores busy 51 % and vector ALU 57 % of the SIMD cycles, at 1.83 GHz.  The better a variant overlapped
// the two, the lower the chip clocked (2.0 GHz with 8 % of the cycles shared, 1.78 with 26 % and four wavefronts per SIMD), so
// what counts is the number of vector instructions per score: one exponential, one addition and half of everything
// else.  128 query tokens, 32/8 heads, 209k
// tokens: 223 us when the GPU was idle before, 250 us back to back (0.88 PFLOP/s of the one product); through the attention
// kernel with one-hot value rows 339 / 369 us.
//
// That is for N(0,1) queries and keys.  A wavefront leaves the interleaved loop for the rest of its split once a row of its 64
// has a first maximum beyond 2^+-40 or a sum beyond 2^80.  A whole ranking, this / one-hot value rows (us): keys 3 / 8 / 12 times
// as large 241 / 360, 255 / 380, 335 / 392 (there every wavefront leaves at its first block); every shot's first key 12 times as
// large (an attention sink) 265 / 387; a mean of 2 common to queries and keys 259 / 357.
//
// Short shots: a segment that ends inside a block costs about 0.25 us a wavefront by factors, whatever its length, and a block of
// many ends about 1.1 us by the one-hot product (short_sums; its 16 fp32 instructions take 1024 cycles).  30000 tokens in
// shots of 1 / 2 / 4 / 6 / 8 / 10, a whole ranking, us; one-hot value rows -- one-hot product -- factors:
//   16 query tokens   240  127   83   63   56   49      89   71   61   58   57   56     270  150   89   69   58   52
//   64 (256 rows)     313  162  107   81   72   64     131  100   87   83   82   80     302  171  111   86   74   68
//   128 (512 rows)    576  280  166  128  116   99     223  158  135  129  125  122     385  215  137  107   95   89
// so the product is taken up to a mean of 6 keys a segment, with two row blocks up to 4.  (With up to 64 query tokens shots of 7 to
// 12 tokens stay 3 to 7 % behind the one-hot value rows; from 15 tokens on this is never slower.)  A segment's end is fetched
// a segment ahead: 1 to 3 % for shots of ten tokens.
#include <type_traits>

#include "mfma_tiles.h"

namespace adapshot {

namespace {
constexpr int kD = 128;
constexpr int kRowBytes = kD * 2;
constexpr int kTileKeys = 64;
constexpr int kTileBytes = kTileKeys * kRowBytes;
constexpr int kBuf = 4;    // K tiles in LDS
constexpr int kWaves = 8;
constexpr int kFrag = 4;   // LDS fragment reads in flight
constexpr int kShortKeys[2] = {6, 4};  // mean keys of a segment up to which the short form is taken: one, two row blocks
constexpr float kLimit = 1.2089258196146292e24f;  // 2^80
constexpr float kUnset = -3.0e38f;                // reference of a row that has seen no key: everything exceeds it
}  // namespace

// SHORT: the form for short shots, which sums the segments that end in a block by matrix instructions (see short_sums).
template <int NR, bool SHORT>
__global__ __launch_bounds__(kWaves * 64) void rank_scores_kernel(RankScoreParams p, int n_row_tiles) {
    constexpr int PASSES = kTileBytes / (kWaves * 1024);  // 1 KB blocks of a tile per wavefront
    __shared__ __attribute__((aligned(16384))) char k_s[kBuf][kTileBytes];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hh = lane >> 5;

    // kv head fastest: workgroups round-robin over the 8 XCDs, so with 8 kv heads an XCD's L2 sees the keys of one
    const int hk = blockIdx.x % p.n_kv_heads;
    const int rest = blockIdx.x / p.n_kv_heads;
    const int row_tile = rest % n_row_tiles, split = rest / n_row_tiles;
    const int g = p.n_q_heads / p.n_kv_heads;
    const int rows = p.t_q * g;
    const int row_base = row_tile * (kWaves * 32 * NR) + wave * 32 * NR;  // first row of this wavefront
    const bool wave_idle = row_base >= rows;
    const int k0 = p.key0 + split * p.keys_per_split;
    const int n_keys = p.n_tok - k0 < p.keys_per_split ? p.n_tok - k0 : p.keys_per_split;  // >= 1
    const int n_tiles = (n_keys + kTileKeys - 1) / kTileKeys;

    // ---- tile loads: wavefront w moves the 1 KB blocks (4 rows) w and w + 8; chunk c of row r goes to c ^ (r & 15).
    // Rows past the last key repeat it; tiles past the last one repeat it whole, so that the number of loads in flight
    // is the same in every iteration.
    const unsigned kv_stride = (unsigned)p.n_kv_heads * kRowBytes;
    const char* const kbase = (const char*)p.k + (int64_t)hk * kRowBytes + (int64_t)k0 * kv_stride;
    unsigned k_loff[PASSES];
#pragma unroll
    for (int ps = 0; ps < PASSES; ++ps) {
        const int r = 4 * (ps * kWaves + wave) + (lane >> 4);
        k_loff[ps] = (unsigned)r * kv_stride + (((lane & 15) ^ (r & 15)) << 4);
    }
    const char* k_tile = kbase;  // next tile to load
    int next_tile = 0;
    auto issue_k = [&](int buf) __attribute__((always_inline)) {
        if (next_tile >= n_tiles - 1) {
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps) {
                const int r = 4 * (ps * kWaves + wave) + (lane >> 4);
                int key = (n_tiles - 1) * kTileKeys + r;
                key = key < n_keys ? key : n_keys - 1;
                load_lds_16(kbase, (unsigned)key * kv_stride + (((lane & 15) ^ (r & 15)) << 4),
                            __builtin_amdgcn_readfirstlane(lds_addr(k_s[buf] + (ps * kWaves + wave) * 1024)));
            }
        } else {
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps)
                load_lds_16(k_tile, k_loff[ps],
                            __builtin_amdgcn_readfirstlane(lds_addr(k_s[buf] + (ps * kWaves + wave) * 1024)));
            k_tile += (unsigned)kTileKeys * kv_stride;
        }
        ++next_tile;
    };

    // ---- Q fragments (B operand): lane holds row l32 of block rb, columns 16*kk + 8*hh .. +7; kk and kk + 4 are rotation
    // partners.  The rows come whole through the LDS that the tiles use afterwards, 32 rows (8 KB) per wavefront at a time.
    bf16x8 qf[NR][8];
    {
        char* const qst = &k_s[0][0] + wave * 8192;
        const int j0 = wave_idle ? 0 : row_base / g;
        const char* qbase = (const char*)p.q + (int64_t)j0 * p.n_q_heads * kRowBytes;
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const int row = row_base + 32 * rb + l32;
            const bool valid = row < rows;
            const int rc = wave_idle ? 0 : valid ? row : rows - 1;
            const int j = rc / g;
            const unsigned qoff = (unsigned)(((j - j0) * p.n_q_heads + hk * g + (rc - j * g)) * kRowBytes);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int rl = 4 * i + (lane >> 4);
                const unsigned off_r = (unsigned)__builtin_amdgcn_ds_bpermute(rl * 4, (int)qoff);
                load_lds_16(qbase, off_r + (((lane & 15) ^ (rl & 15)) << 4),
                            __builtin_amdgcn_readfirstlane(lds_addr(qst + i * 1024)));
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            const int64_t a = p.q_pos0 + j;
            const float2* th = p.tab_hi + (a >> kRopeLoBits) * (kD / 2);
            const float2* tl = p.tab_lo + (a & (kRopeLo - 1)) * (kD / 2);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                u32x4 x1 = *(const u32x4*)(qst + l32 * 256 + (((2 * kk + hh) ^ (l32 & 15)) << 4));
                u32x4 x2 = *(const u32x4*)(qst + l32 * 256 + (((2 * (kk + 4) + hh) ^ (l32 & 15)) << 4));
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const f32x4 h = *(const f32x4*)(th + 16 * kk + 8 * hh + 2 * w), l = *(const f32x4*)(tl + 16 * kk + 8 * hh + 2 * w);
                    const float c0 = h[0] * l[0] - h[1] * l[1], s0 = h[1] * l[0] + h[0] * l[1];
                    const float c1 = h[2] * l[2] - h[3] * l[3], s1 = h[3] * l[2] + h[2] * l[3];
                    const float a1l = __uint_as_float(x1[w] << 16), a1h = __uint_as_float(x1[w] & 0xffff0000u);
                    const float a2l = __uint_as_float(x2[w] << 16), a2h = __uint_as_float(x2[w] & 0xffff0000u);
                    x1[w] = pack2_bf16((a1l * c0 - a2l * s0) * p.q_scale, (a1h * c1 - a2h * s1) * p.q_scale);
                    x2[w] = pack2_bf16((a2l * c0 + a1l * s0) * p.q_scale, (a2h * c1 + a1h * s1) * p.q_scale);
                }
                const u32x4 zero = {0u, 0u, 0u, 0u};
                qf[rb][kk] = __builtin_bit_cast(bf16x8, valid ? x1 : zero);
                qf[rb][kk + 4] = __builtin_bit_cast(bf16x8, valid ? x2 : zero);
            }
            // read before the next 32 rows arrive, and rotated here, not where the compiler would move it: into the loops
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(qf[rb][0]), "+v"(qf[rb][1]), "+v"(qf[rb][2]), "+v"(qf[rb][3]), "+v"(qf[rb][4]),
                           "+v"(qf[rb][5]), "+v"(qf[rb][6]), "+v"(qf[rb][7])
                         :
                         : "memory");
        }
    }
    __syncthreads();
    issue_k(0);
    issue_k(1);
    issue_k(2);

    // ---- segments of this split, their ends relative to k0 (scalar loads: the vector memory counter belongs to the tiles)
    typedef const __attribute__((address_space(4))) int32_t* table_t;
    const table_t seg_end = (table_t)(uintptr_t)p.seg_end, seg0 = (table_t)(uintptr_t)p.split_seg0;
    const int seg_first = seg0[split], seg_stop = seg0[split + 1];
    int seg = seg_first;
    // end of the segment (relative to k0; behind the split's last: none) -- `after`, the next one's, is fetched a segment ahead
    auto end_of = [&](int q) __attribute__((always_inline)) -> int {
        const int e = seg_end[q < seg_stop ? q : seg_stop - 1] - k0;
        return q < seg_stop ? e : 0x7fffffff;
    };
    int next_end = end_of(seg), after = end_of(seg + 1);
    const int64_t n_pairs = (int64_t)rows * p.n_kv_heads;
    const int my_row = row_base + (NR == 2 ? lane : l32);  // the row this lane stores
    const bool store_on = my_row < rows && (NR == 2 || hh == 0);
    float* const part = p.part + (int64_t)hk * rows + my_row;

    // Row i of the product's A operand is key 8 (i/8) + 2 (i%4) + (i/4)%2 of the block, so that register r of a result
    // holds key 2r + l/32: a segment's end falls between the same two registers in all lanes, or into one register.
    const int k_row = (l32 & 24) + 2 * (l32 & 3) + ((l32 >> 2) & 1);
    unsigned ka[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) ka[kk] = lds_addr(&k_s[0][0]) + (unsigned)(k_row * kRowBytes + (((2 * kk + hh) ^ (k_row & 15)) << 4));
    typedef __attribute__((address_space(3))) char lds_char;
    lds_char* kp[8];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) kp[kk] = (lds_char*)(uintptr_t)ka[kk];

    typedef f32x16 block_t[NR];  // the scores of 32 keys and 32 * NR rows
    block_t s0, s1;
    float m[NR], acc[NR];
    float l_run = 0.f;  // of my_row
    float l_short[NR];  // SHORT: of row l32 of every row block, what this half of the lanes has stored
#pragma unroll
    for (int rb = 0; rb < NR; ++rb) {
        m[rb] = 0.f;
        acc[rb] = 0.f;
        l_short[rb] = 0.f;
    }

    // Pointers to the fragments of tile t
    auto point = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) kp[kk] = (lds_char*)(uintptr_t)(ka[kk] + (unsigned)(t & (kBuf - 1)) * kTileBytes);
    };
    // s = K . Q^T of block kb; EXPS: x = 2^x meanwhile, two exponentials behind every product
    auto s_phase = [&](int kb, block_t& s, block_t& x, auto with_exps) __attribute__((always_inline)) {
        auto frag = [&](int kk) __attribute__((always_inline)) -> bf16x8 {
            return __builtin_bit_cast(bf16x8, *(const __attribute__((address_space(3))) u32x4*)(kp[kk] + kb * (32 * kRowBytes)));
        };
        const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        bf16x8 fr[kFrag];
#pragma unroll
        for (int i = 0; i < kFrag; ++i) fr[i] = frag(i);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
            const bf16x8 a = fr[kk % kFrag];
            if (kk + kFrag < 8) fr[kk % kFrag] = frag(kk + kFrag);
#pragma unroll
            for (int rb = 0; rb < NR; ++rb)
                s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[rb][kk], kk == 0 ? zero : s[rb], 0, 0, 0);
            if constexpr (decltype(with_exps)::value) {
#pragma unroll
                for (int rb = 0; rb < NR; ++rb) {
                    x[rb][2 * kk] = __builtin_amdgcn_exp2f(x[rb][2 * kk]);
                    x[rb][2 * kk + 1] = __builtin_amdgcn_exp2f(x[rb][2 * kk + 1]);
                }
            }
        }
        __builtin_amdgcn_sched_group_barrier(0x100, kFrag, 0);
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if constexpr (decltype(with_exps)::value) __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
            }
            if (kk + kFrag < 8) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
    };
    // The segment that ends here leaves: v = the sums of the lane's own half of the keys.
    auto flush = [&](const float (&v)[NR]) __attribute__((always_inline)) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[NR - 1]), false, false);
        const float x = __uint_as_float(r[0]) + __uint_as_float(r[1]);
        l_run += x;
        if (store_on) part[(int64_t)seg * n_pairs] = x;
    };
    auto exps_moved = [&](block_t& s) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < NR; ++rb)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[rb][r] = __builtin_amdgcn_exp2f(s[rb][r] - m[rb]);
    };
    // a = acc + the sums of the whole block
    auto whole_sums = [&](const block_t& s, float (&a)[NR]) __attribute__((always_inline)) {
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            float u = acc[rb] + s[rb][0], v = s[rb][1];
#pragma unroll
            for (int r = 2; r < 16; r += 2) {
                u += s[rb][r];
                v += s[rb][r + 1];
            }
            a[rb] = u + v;
        }
    };
    // Sums of the block's keys before `end` (1..32) into a, from it on into b.  Whole registers go to one side by scalar 0 / 1
    // factors; the register that an odd end cuts goes to either side by lane half.
    auto split_sums = [&](const block_t& s, int end, float (&a)[NR], float (&b)[NR]) __attribute__((always_inline)) {
        const int rs = end >> 1;
        const bool odd = end & 1;
        const int rb0 = rs + (odd ? 1 : 0);
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const f32x16 v = s[rb];
            const float x = odd ? v[rs & 15] : 0.f;
            a[rb] = hh ? 0.f : x;
            b[rb] = hh ? x : 0.f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float f = __uint_as_float(__builtin_amdgcn_readfirstlane(r < rs ? 0x3f800000u : 0u));
            const float h = __uint_as_float(__builtin_amdgcn_readfirstlane(r >= rb0 ? 0x3f800000u : 0u));
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) {
                a[rb] = fmaf(s[rb][r], f, a[rb]);
                b[rb] = fmaf(s[rb][r], h, b[rb]);
            }
        }
    };
    auto row_max = [&](const block_t& s, int rb) __attribute__((always_inline)) -> float {
        // The first maximum is no inline assembly: it waits for the product, as the compiler sees to.
        float mx = fmaxf(s[rb][15], s[rb][0]);
#pragma unroll
        for (int r = 1; r < 15; r += 2) mx = max3(mx, s[rb][r], s[rb][r + 1]);
        return max_xhalf(mx);
    };
    // What exceeds its row's reference by far moves it, and what the split has summed so far is scaled; s is computed again.
    auto move_references = [&](int t, int kb, block_t& s) __attribute__((always_inline)) {
        point(t);
        s_phase(kb, s, s, std::false_type{});
        float alpha[NR];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const float mx = row_max(s, rb);
            const float m_new = mx - m[rb] > 40.f ? mx : m[rb];
            alpha[rb] = __builtin_amdgcn_exp2f(m[rb] - m_new);
            m[rb] = m_new;
            acc[rb] *= alpha[rb];
            if (SHORT) l_short[rb] *= alpha[rb];
        }
        const float al = NR == 2 && hh ? alpha[NR - 1] : alpha[0];
        l_run *= al;
        if (store_on)
            for (int q = seg_first; q < seg; ++q) part[(int64_t)q * n_pairs] *= al;
        exps_moved(s);
    };
    auto is_over = [&](const float (&x)[NR]) __attribute__((always_inline)) -> bool {
        bool o = !(x[0] <= kLimit);  // (also where an overflow has met a factor 0)
        if (NR == 2) o |= !(x[NR - 1] <= kLimit);
        return __builtin_amdgcn_ballot_w64(o) != 0;
    };
    // The segments that end in the block, all of them at once: sums = one-hot . P with v_mfma_f32_32x32x2_f32.  Register r of a
    // block is the B operand as it stands (lane = row, key 2r + l/32); the A operand's lane holds 1 where that key belongs to
    // the segment l%32 of the block.  Products with 0 and 1 and sums in fp32.  Row i of the result, in the lanes of half
    // (i/4)%2, is the sum of the block's segment i; the one behind the last end is carried on.
    auto short_sums = [&](unsigned ends, const block_t& s) __attribute__((always_inline)) {
        constexpr int CH = NR == 1 ? 2 : 1;  // chains of products: two row blocks are two already
        const int n_end = __builtin_popcount(ends);  // >= 1
        f32x16 d[NR][CH];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
#pragma unroll
            for (int c = 0; c < CH; ++c)
                d[rb][c] = f32x16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            const float c = sum_xhalf(acc[rb]);  // what the first segment has from the blocks before
            d[rb][0][0] = hh ? 0.f : c;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int before = __builtin_popcount(__builtin_amdgcn_ubfe(ends, 0, 2 * r + hh));  // the key's segment
            const float one = before == l32 ? 1.f : 0.f;
#pragma unroll
            for (int rb = 0; rb < NR; ++rb)
                d[rb][r % CH] = __builtin_amdgcn_mfma_f32_32x32x2f32(one, s[rb][r], d[rb][r % CH], 0, 0, 0);
        }
        if (CH == 2) d[0][0] += d[0][CH - 1];
        float* out[NR];
        int lim[NR];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const int row = row_base + 32 * rb + l32;
            out[rb] = p.part + (int64_t)(seg + 4 * hh) * n_pairs + (int64_t)hk * rows + row;
            lim[rb] = row < rows ? n_end - 4 * hh : 0;
        }
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4)
            if (8 * i4 < n_end) {
#pragma unroll
                for (int i = 4 * i4; i < 4 * i4 + 4; ++i) {
                    const int first = 8 * i4 + (i & 3);
#pragma unroll
                    for (int rb = 0; rb < NR; ++rb)
                        if (first < lim[rb]) {
                            l_short[rb] += d[rb][0][i];
                            out[rb][first * n_pairs] = d[rb][0][i];
                        }
                }
            }
        const int i_rest = (n_end >> 3) * 4 + (n_end & 3);
        const bool here = n_end < 32 && hh == ((n_end >> 2) & 1);
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const f32x16 v = d[rb][0];
            const float x = v[i_rest & 15];
            acc[rb] = here ? x : 0.f;
        }
        seg += n_end;
    };
    // The bits of the segment ends in the block that begins at key_b: 0 behind the last key
    auto block_ends = [&](int key_b) __attribute__((always_inline)) -> unsigned {
        const int b = key_b < n_keys ? key_b : 0;
        const unsigned w = ((table_t)(uintptr_t)p.end_bits)[(split * p.keys_per_split + b) >> 5];
        return key_b < n_keys ? w : 0u;
    };
    unsigned ends_here = SHORT ? block_ends(0) : 0u;  // of the next block to sum, fetched a block ahead
    // Sums of a block whose exponentials are in s.  `moved`: references other than 0 are in use, and moved where that is
    // needed; without it the result says whether the sums were in range, and nothing has changed where they were not.
    auto sums = [&](int t, int kb, block_t& s, bool moved) __attribute__((always_inline)) -> bool {
        const int key_b = t * kTileKeys + kb * 32;  // first key of the block
        if constexpr (SHORT) {
            float a[NR];
            whole_sums(s, a);
            if (__builtin_expect(is_over(a), 0)) {
                if (!moved) return false;
                move_references(t, kb, s);
                whole_sums(s, a);
            }
            const unsigned ends = ends_here;
            ends_here = block_ends(key_b + 32);
            if (ends) {
                short_sums(ends, s);
            } else {
#pragma unroll
                for (int rb = 0; rb < NR; ++rb) acc[rb] = a[rb];
            }
            return true;
        }
        // a: the sum of the segment that ends here (or with the whole block, nothing ending), b: of what lies behind it
        float a[NR], b[NR];
        if (__builtin_expect(next_end > key_b + 32, 1)) {
            whole_sums(s, a);
            if (__builtin_expect(is_over(a), 0)) {
                if (!moved) return false;
                move_references(t, kb, s);
                whole_sums(s, a);
            }
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) acc[rb] = a[rb];
            return true;
        }
        split_sums(s, next_end - key_b, a, b);
        float c[NR];
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) c[rb] = acc[rb] + (a[rb] + b[rb]);
        if (__builtin_expect(is_over(c), 0)) {
            if (!moved) return false;
            move_references(t, kb, s);
            split_sums(s, next_end - key_b, a, b);
        }
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) a[rb] += acc[rb];
        flush(a);
        ++seg;
        int done = next_end - key_b;  // keys of the block whose segments have left
        next_end = after;
        after = end_of(seg + 1);
        while (next_end <= key_b + 32) {  // short segments that begin and end in this block: 0 / 1 factors
            const float lo = (float)(done - hh), hi = (float)(next_end - key_b - hh);
#pragma unroll
            for (int rb = 0; rb < NR; ++rb) a[rb] = b[rb] = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float before = __builtin_amdgcn_fmed3f(hi - (float)(2 * r), 0.f, 1.f);  // 1: the key lies before the end
                const float f = before - __builtin_amdgcn_fmed3f(lo - (float)(2 * r), 0.f, 1.f);
#pragma unroll
                for (int rb = 0; rb < NR; ++rb) {
                    a[rb] = fmaf(f, s[rb][r], a[rb]);
                    b[rb] = fmaf(1.f - before, s[rb][r], b[rb]);
                }
            }
            flush(a);
            ++seg;
            done = next_end - key_b;
            next_end = after;
            after = end_of(seg + 1);
        }
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) acc[rb] = b[rb];
        return true;
    };
    // The products of tile t are done in every wavefront: K(t+1) has landed (K(t+2) may stay in flight, and segment sums on
    // their way out only make the wait stricter), and K(t-1), kept for second looks until now, makes room for K(t+3).
    static_assert(PASSES == 2, "vmcnt immediates");
    auto next_tile_ready = [&](int t) __attribute__((always_inline)) {
        asm volatile("s_waitcnt vmcnt(2) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        issue_k((t + 3) & (kBuf - 1));
    };

    asm volatile("s_waitcnt vmcnt(4) lgkmcnt(0)\n\ts_barrier" ::: "memory");  // K(0)
    if (wave_idle) {
        for (int t = 0; t < n_tiles; ++t) next_tile_ready(t);
    } else {
        point(0);
        s_phase(0, s0, s0, std::false_type{});
        bool moved = false;
#pragma unroll
        for (int rb = 0; rb < NR; ++rb) {
            const float mx = row_max(s0, rb);
            m[rb] = fabsf(mx) < 40.f ? 0.f : fmaxf(mx, kUnset);
            moved |= m[rb] != 0.f;
        }
        moved = __builtin_amdgcn_ballot_w64(moved) != 0;
        int t = 0, first_kb = 0;
        if (!moved) {
            for (; t < n_tiles; ++t) {
                s_phase(1, s1, s0, std::true_type{});
                if (!sums(t, 0, s0, false)) break;
                next_tile_ready(t);
                point(t + 1);
                s_phase(0, s0, s1, std::true_type{});  // past the end: of a repeated tile, unused
                if (!sums(t, 1, s1, false)) {
                    first_kb = 1;
                    break;
                }
            }
        }
        for (; t < n_tiles; ++t) {  // references other than 0
            point(t);
            if (first_kb == 0) {
                s_phase(0, s0, s0, std::false_type{});
                exps_moved(s0);
                sums(t, 0, s0, true);
                point(t);
                s_phase(1, s1, s1, std::false_type{});
                next_tile_ready(t);
            } else {
                s_phase(1, s1, s1, std::false_type{});
                first_kb = 0;
            }
            exps_moved(s1);
            sums(t, 1, s1, true);
        }
    }
    if (SHORT) {
        const float l0 = sum_xhalf(l_short[0]), l1 = sum_xhalf(l_short[NR - 1]);
        l_run += NR == 2 && hh ? l1 : l0;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the loads past the end must land before LDS is released
    if (!wave_idle && store_on)
        p.part_ml[(int64_t)split * n_pairs + (int64_t)hk * rows + my_row] = make_float2(NR == 2 && hh ? m[NR - 1] : m[0], l_run);
}

hipError_t launch_rank_scores(const RankScoreParams& p, hipStream_t stream) {
    const int rows = p.t_q * (p.n_q_heads / p.n_kv_heads);
    // Two row blocks per wavefront halve the LDS reads per product (512 rows: 223 us against 230 us in two tiles of 256); up
    // to 256 rows they would leave wavefronts idle.
    const int tile = rows > 256 ? 512 : 256;
    const int n_row_tiles = (rows + tile - 1) / tile;
    const unsigned blocks = (unsigned)(p.n_kv_heads * n_row_tiles * p.n_split);
    if (blocks == 0) return hipSuccess;
    const bool short_segments = (int64_t)p.n_seg * kShortKeys[tile == 512] >= p.n_tok - p.key0;
    if (tile == 512) {
        if (short_segments) launch_kernel((rank_scores_kernel<2, true>), dim3(blocks), dim3(kWaves * 64), stream, p, n_row_tiles);
        else launch_kernel((rank_scores_kernel<2, false>), dim3(blocks), dim3(kWaves * 64), stream, p, n_row_tiles);
    } else {
        if (short_segments) launch_kernel((rank_scores_kernel<1, true>), dim3(blocks), dim3(kWaves * 64), stream, p, n_row_tiles);
        else launch_kernel((rank_scores_kernel<1, false>), dim3(blocks), dim3(kWaves * 64), stream, p, n_row_tiles);
    }
    return hipGetLastError();
}

}  // namespace adapshot
