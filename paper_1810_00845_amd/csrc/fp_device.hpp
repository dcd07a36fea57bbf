// Device helpers shared by the fp64 kernels (ntt_fp.hip, convert_fp.hip): scalar table reads, buffer-resource
// accesses, wave-local ordering of LDS traffic, the NTT-order automorphism.
#pragma once
#include "hisa_internal.hpp"
#include "fparith.hpp"

// Read-only tables indexed by wave-uniform values go through the constant address space, which makes the
// compiler use scalar loads (SGPR results, batched, off the vector memory path).  Vector loads of uniform
// addresses were each followed by a wait and cost the kernel dozens of exposed memory latencies.
typedef const __attribute__((address_space(4))) double* cdouble_ptr;
__device__ __forceinline__ cdouble_ptr as_const(const double* p) { return (cdouble_ptr)(unsigned long long)p; }

// Per-lane global accesses go through buffer resources: one (base, size) descriptor per object in scalar registers,
// the lane's byte offset in ONE vector register per mapping and the row's offset in a scalar register or the
// instruction.  Plain pointers cost one or two 64-bit vector additions per access (hundreds per task) and a register
// pair each; this form costs none, and the hardware drops any access beyond `bytes` instead of faulting.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u64 bload(rsrc_t r, uint32_t lane_off, uint32_t row_off) {
    const u32x2_t d = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)row_off, 0);
    return ((u64)d.y << 32) | d.x;
}
// the same, bypassing the CU's L1 (data that another point in time of this workgroup wrote)
__device__ __forceinline__ u64 bload_glc(rsrc_t r, uint32_t lane_off, uint32_t row_off) {
    const u32x2_t d = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)row_off, 1);
    return ((u64)d.y << 32) | d.x;
}
__device__ __forceinline__ double bloadf(rsrc_t r, uint32_t lane_off, uint32_t row_off) {
    return __longlong_as_double((long long)bload(r, lane_off, row_off));
}
__device__ __forceinline__ void bstore(rsrc_t r, uint32_t lane_off, uint32_t row_off, u64 x) {
    u32x2_t d;
    d.x = (uint32_t)x; d.y = (uint32_t)(x >> 32);
    __builtin_amdgcn_raw_buffer_store_b64(d, r, (int)lane_off, (int)row_off, 0);
}
__device__ __forceinline__ void bstoref(rsrc_t r, uint32_t lane_off, uint32_t row_off, double x) {
    bstore(r, lane_off, row_off, (u64)__double_as_longlong(x));
}

// keeps the compiler from moving instructions across this point (loads issued in batches stay batches)
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

__device__ __forceinline__ uint32_t lo32(double v) { return (uint32_t)__double_as_longlong(v); }
__device__ __forceinline__ uint32_t hi32(double v) { return (uint32_t)((u64)__double_as_longlong(v) >> 32); }
__device__ __forceinline__ double mk64(uint32_t lo, uint32_t hi) { return __longlong_as_double((long long)(((u64)hi << 32) | lo)); }

// Synchronisation between the writes and the reads of a transpose.  A transpose inside one wave needs no hardware
// barrier: a wave's LDS instructions execute in issue order, so its reads see its earlier writes and its later
// writes cannot overtake its earlier reads; the compiler only has to keep that order.
template <bool LOCAL>
__device__ __forceinline__ void xchg_sync() {
    if (LOCAL) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    } else {
        __syncthreads();
    }
}

__device__ __forceinline__ uint32_t galois_src_fp(uint32_t i, u64 g, int log_n) {
    const uint32_t mask = (2u << log_n) - 1;
    const uint32_t e = 2 * (__brev(i) >> (32 - log_n)) + 1;
    const uint32_t e2 = (uint32_t)((u64)e * g) & mask;
    return __brev((e2 - 1) >> 1) >> (32 - log_n);
}

