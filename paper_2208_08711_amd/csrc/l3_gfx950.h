/*
 * gfx950 primitives of the L3 kernels: vector and address-space types, lane shifts, packed
 * 16-bit operations, LDS addressing by 32-bit address, register pinning.  Everything in the
 * decoder and the encoder that names the target sits here or is an amdgcn builtin; their own
 * logic (l3_kernel_parts.h, l3_device.hip, l3_encode.hip) is written on top of these names.  (A host
 * build of the kernels for the sanitizers replaces this file alone: tests/native/kernel_cpu.)
 * Device code only; every translation unit gets its own copy.
 */
#ifndef L3_GFX950_H
#define L3_GFX950_H

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef u32x3 u32x3_any __attribute__((aligned(1)));      /* any byte alignment */
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_any __attribute__((aligned(1)));

typedef __attribute__((address_space(1))) const u32x4 global_const_u32x4;
typedef __attribute__((address_space(1))) const u32_any global_const_u32_any;
typedef __attribute__((address_space(1))) u32x3_any global_u32x3_any;
typedef __attribute__((address_space(1))) u32_any global_u32_any;
typedef __attribute__((address_space(1))) u32x2_any global_u32x2_any;
typedef __attribute__((address_space(1))) const u32x3_any global_const_u32x3_any;
typedef u32x4 u32x4_any __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) u32x4 global_u32x4;
typedef __attribute__((address_space(1))) u32x4_any global_u32x4_any;
typedef __attribute__((address_space(1))) const uint8_t global_const_u8;
typedef __attribute__((address_space(1))) uint8_t global_u8;
typedef uint16_t u16_any __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) u16_any global_u16_any;

/* 12 bytes at any alignment, and no more */
__device__ __forceinline__ u32x3 load_u32x3(global_const_u8* p) { return *reinterpret_cast<global_const_u32x3_any*>(p); }

__device__ __forceinline__ uint32_t dpp_from_lower_lane(uint32_t v) {   /* lane i <- lane i-1, lane 0 <- 0 */
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t dpp_from_upper_lane(uint32_t v) {   /* lane i <- lane i+1, lane 63 <- 0 */
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
}

/* What follows is written with builtins where these become the instruction named, and not as
 * inline assembly: behind that the compiler puts a wait state (s_nop) ahead of every use. */

/* Both 16-bit halves of v shifted right by the low half of `by` (modulo 16): v_pk_lshrrev_b16. */
__device__ __forceinline__ uint32_t pk_lshr_b16_by_low(uint32_t by, uint32_t v) {
    const unsigned short s = (unsigned short)(by & 15u);
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, v) >> (u16x2){s, s}));
}
/* a * (low half of b) + c in both 16-bit halves, modulo 2^16: v_pk_mad_u16. */
__device__ __forceinline__ uint32_t pk_mad_u16_by_low(uint32_t a, uint32_t b, uint32_t c) {
    const unsigned short f = (unsigned short)b;
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) * (u16x2){f, f} + __builtin_bit_cast(u16x2, c)));
}
/* Both 16-bit halves: the low half of v shifted right by the halves of `by` (below 16; a value
 * that the compiler does not know, or it shifts before it copies): v_pk_lshrrev_b16. */
__device__ __forceinline__ uint32_t low_b16_lshr_twice(uint32_t by, uint32_t v) {
    const unsigned short low = (unsigned short)v;
    return __builtin_bit_cast(uint32_t, (u16x2)((u16x2){low, low} >> __builtin_bit_cast(u16x2, by)));
}

/* Packed 16-bit floats, used as exact integers.  Smallest and largest of three
 * (v_pk_minimum3_f16, v_pk_maximum3_f16): */
__device__ __forceinline__ uint32_t pk_min3_f16(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_minimum(
        __builtin_elementwise_minimum(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b)), __builtin_bit_cast(f16x2, c)));
}
__device__ __forceinline__ uint32_t pk_max3_f16(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_maximum(
        __builtin_elementwise_maximum(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b)), __builtin_bit_cast(f16x2, c)));
}
__device__ __forceinline__ uint32_t pk_add_f16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (f16x2)(__builtin_bit_cast(f16x2, a) + __builtin_bit_cast(f16x2, b)));
}
__device__ __forceinline__ uint32_t pk_sub_f16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (f16x2)(__builtin_bit_cast(f16x2, a) - __builtin_bit_cast(f16x2, b)));
}
/* c + a * b and c - a * b, rounded once (v_pk_fma_f16) */
__device__ __forceinline__ uint32_t pk_fma_f16(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b),
                                                                  __builtin_bit_cast(f16x2, c)));
}
__device__ __forceinline__ uint32_t pk_fnma_f16(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(-__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b),
                                                                  __builtin_bit_cast(f16x2, c)));
}
/* 2a - b, held between 0 and 1 (one v_pk_fma_f16 with clamp): of whole numbers, 1 where 2a > b
 * and 0 elsewhere */
__device__ __forceinline__ uint32_t pk_twice_exceeds_f16(uint32_t a, uint32_t b) {
    const f16x2 zero = {0, 0}, one = {1, 1}, two = {2, 2};
    const f16x2 d = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, a), two, -__builtin_bit_cast(f16x2, b));
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_elementwise_max(d, zero), one));
}
/* One instruction also where the compiler would keep the inner maximum for another path. */
__device__ __forceinline__ uint32_t max3_u32(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_max3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

/* true in every lane if `mine` is true in any lane of the wave */
__device__ __forceinline__ bool wave_any(bool mine) { return __builtin_amdgcn_ballot_w64(mine) != 0; }

/* ---- LDS by 32-bit address ------------------------------------------------ */

typedef __attribute__((address_space(3))) const uint32_t lds_const_u32;
struct LdsPair { uint32_t lo, hi; };
__device__ __forceinline__ uint32_t lds_address_of(const uint32_t* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const uint32_t*)p;
}
/* the two consecutive words at LDS address `where` (one ds_read2_b32) */
__device__ __forceinline__ LdsPair lds_read_pair(uint32_t where) {
    lds_const_u32* p = reinterpret_cast<lds_const_u32*>(where);
    LdsPair v;
    v.lo = p[0];
    v.hi = p[1];
    return v;
}

__device__ __forceinline__ uint32_t lds_read_u32(uint32_t where) {
    return *reinterpret_cast<lds_const_u32*>(where);
}
__device__ __forceinline__ u32x2 lds_read_u32x2(uint32_t where) {      /* 8-byte aligned */
    return *reinterpret_cast<__attribute__((address_space(3))) const u32x2*>(where);
}
__device__ __forceinline__ u32x4 lds_read_u32x4(uint32_t where) {      /* 16-byte aligned */
    return *reinterpret_cast<__attribute__((address_space(3))) const u32x4*>(where);
}
__device__ __forceinline__ void lds_write_u32x2(uint32_t where, u32x2 v) {
    *reinterpret_cast<__attribute__((address_space(3))) u32x2*>(where) = v;
}
__device__ __forceinline__ void lds_write_u32x4(uint32_t where, u32x4 v) {
    *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(where) = v;
}

/* ORs lo and hi into the two consecutive words at LDS address `where`, each atomically among the workgroup's threads */
__device__ __forceinline__ void lds_or_pair(uint32_t where, uint32_t lo, uint32_t hi) {
    __attribute__((address_space(3))) uint32_t* cell = reinterpret_cast<__attribute__((address_space(3))) uint32_t*>(where);
    __hip_atomic_fetch_or(cell, lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_fetch_or(cell + 1, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

/* ---- words that workgroups of a launch share -------------------------------- */

/* Each of these is one access that all workgroups of the GPU see alike; none orders other accesses. */
__device__ __forceinline__ uint64_t agent_load_u64(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_store_u64(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t agent_exchange_u32(uint32_t* p, uint32_t v) {
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t agent_exchange_u64(uint64_t* p, uint64_t v) {
    return __hip_atomic_exchange(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t agent_add_u64(uint64_t* p, uint64_t v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

/* LDS of the size that the launch gives */
#define L3_DYNAMIC_LDS(type, name) extern __shared__ type name[]

/* ---- keeping a value where it is ------------------------------------------ */

/* The value becomes opaque to the optimiser and stays in a vector (scalar) register: used
 * where the compiler would otherwise widen, rematerialise or reload it at a bad place. */
#define L3_KEEP_VGPR(x) asm volatile("" : "+v"(x))
/* memory accesses behind this follow the one that x comes from */
#define L3_WAIT_FOR(x) asm volatile("" : "+v"(x) : : "memory")
#define L3_KEEP_SGPR(x) asm volatile("" : "+s"(x))

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

#endif
