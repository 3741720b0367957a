// Device helpers shared by the matrix-core kernels (attention, streaming attention, ranking).
#pragma once
#include "adapshot_internal.h"

namespace adapshot {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// max / sum over the two lanes l and l^32 without going through LDS
__device__ __forceinline__ float max_xhalf(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xhalf(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// max / sum over the 64 lanes, the same in every lane
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    const int u = (int)__float_as_uint(v);
    return __uint_as_float((unsigned)__builtin_amdgcn_update_dpp(u, u, CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float max_xrow(float v) {  // lanes l and l^16
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_xrow(float v) {
    const unsigned u = __float_as_uint(v);
    const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppHalfMirror = 0x141, kDppMirror = 0x140;  // quad_perm, row_half_mirror, row_mirror
__device__ __forceinline__ float wave_max(float v) {
    v = fmaxf(v, dpp<kDppXor1>(v));
    v = fmaxf(v, dpp<kDppXor2>(v));
    v = fmaxf(v, dpp<kDppHalfMirror>(v));
    v = fmaxf(v, dpp<kDppMirror>(v));
    return max_xhalf(max_xrow(v));
}
__device__ __forceinline__ float wave_sum(float v) {
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppMirror>(v);
    return sum_xhalf(sum_xrow(v));
}

__device__ __forceinline__ unsigned pack2_bf16(float lo, float hi) {
    f32x2 f = {lo, hi};
    bf16x2 b = __builtin_convertvector(f, bf16x2);  // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(unsigned, b);
}

// max of three in one instruction.  fmaxf() chains compile to twice as many instructions because every
// input is first canonicalised; the scores here are MFMA outputs or -inf, never signalling NaNs.
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// ---- buffer accesses: a base and a size in scalar registers, a 32-bit byte offset per lane.  Reads past the size return zero.
constexpr int kCacheDevice = 16;  // past the L2 of the workgroup's XCD, for data that other workgroups of the launch write or read
typedef __amdgpu_buffer_rsrc_t buf_rsrc;
__device__ __forceinline__ buf_rsrc make_buffer(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);  // raw, 32-bit data
}
template <int CACHE = 0>
__device__ __forceinline__ u32x4 buf_load_16(buf_rsrc r, unsigned off) {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, CACHE));
}
template <int CACHE = 0>
__device__ __forceinline__ u32x2 buf_load_8(buf_rsrc r, unsigned off) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, CACHE));
}
__device__ __forceinline__ unsigned buf_load_4(buf_rsrc r, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0); }
__device__ __forceinline__ unsigned short buf_load_2(buf_rsrc r, unsigned off) { return __builtin_amdgcn_raw_buffer_load_b16(r, (int)off, 0, 0); }
// 16 bytes per lane straight into LDS: lane l's land at dst + 16*l (dst is wave-uniform).  The compiler knows these loads: it waits for
// those into an array before it reads from that array, and for no others.
__device__ __forceinline__ void buf_load_lds_16(buf_rsrc r, char* dst, unsigned off) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void*)dst, 16, (int)off, 0, 0, 0);
}
template <int CACHE = 0>
__device__ __forceinline__ void buf_store_16(buf_rsrc r, unsigned off, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)off, 0, CACHE);
}

// 16 bytes per lane from global memory straight into LDS: lane l's data lands at lds_base + 16*l
// (lds_base is wave-uniform and goes through M0; the source is a uniform base plus a 32-bit lane offset).
// Issued as inline assembly so that the key loop keeps control of the wait counters: the loads complete
// in order and are awaited with vmcnt in barrier_keep_one_group(), tiles after they were issued.
// NT marks the data as read once (the instruction's non-temporal bit): a launch whose workgroups stream their
// context with one or two working wavefronts is bound by the memory path, and tiles that are not kept in the L2
// for a reader that never comes move 10 % faster (5.9 -> 6.45 TB/s for the bare tile stream of a decode step).
template <bool NT = false>
__device__ __forceinline__ void load_lds_16(const char* gbase, unsigned goff, unsigned lds_base) {
    unsigned saved_m0;
    if (NT)
        asm volatile(
            "s_mov_b32 %0, m0\n\t"
            "s_mov_b32 m0, %3\n\t"
            "global_load_lds_dwordx4 %1, %2 nt\n\t"
            "s_mov_b32 m0, %0"
            : "=&s"(saved_m0)
            : "v"(goff), "s"(gbase), "s"(lds_base)
            : "memory");
    else
        asm volatile(
            "s_mov_b32 %0, m0\n\t"
            "s_mov_b32 m0, %3\n\t"
            "global_load_lds_dwordx4 %1, %2\n\t"
            "s_mov_b32 m0, %0"
            : "=&s"(saved_m0)
            : "v"(goff), "s"(gbase), "s"(lds_base)
            : "memory");
}
__device__ __forceinline__ unsigned lds_addr(const void* p) {
    return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

}  // namespace adapshot
