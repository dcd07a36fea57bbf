// Device helpers shared by the transforms (ntt_fp.hip, convert_fp.hip, convert_int.hip): scalar table reads, buffer-resource
// accesses, wave-local ordering of LDS traffic, the NTT-order automorphism, rows by one wave and by four.
#pragma once
#include <algorithm>
#include <type_traits>

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

// two neighbouring words, 16 bytes
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void bload2(rsrc_t r, uint32_t lane_off, uint32_t row_off, u64& x, u64& y) {
    const u32x4_t d = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)row_off, 0);
    x = ((u64)d.y << 32) | d.x;
    y = ((u64)d.w << 32) | d.z;
}
__device__ __forceinline__ void bload2(rsrc_t r, uint32_t lane_off, uint32_t row_off, double& x, double& y) {
    u64 a, b;
    bload2(r, lane_off, row_off, a, b);
    x = __longlong_as_double((long long)a);
    y = __longlong_as_double((long long)b);
}
__device__ __forceinline__ void bstore2(rsrc_t r, uint32_t lane_off, uint32_t row_off, u64 x, u64 y) {
    const u32x4_t d = {(uint32_t)x, (uint32_t)(x >> 32), (uint32_t)y, (uint32_t)(y >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(d, r, (int)lane_off, (int)row_off, 0);
}
__device__ __forceinline__ void bstore2(rsrc_t r, uint32_t lane_off, uint32_t row_off, double x, double y) {
    bstore2(r, lane_off, row_off, (u64)__double_as_longlong(x), (u64)__double_as_longlong(y));
}

// The keys of a launch (up to 32 rotations) that reads each of them once pass the caches by (nontemporal) when the last-level cache, 256 MB,
// will not hold them until the next call: they only displace the digits and what the next launch reads.  Rotations of one ciphertext, us, kept /
// passed by: N = 2^14, 12 limbs, 189 MB of keys (15 rotations) 101 / 106, 227 MB 124 / 122, 302 MB 153 / 142; N = 2^15, 20 limbs, 213 MB
// 146 / 143, 340 MB 191 / 175, 680 MB 344 / 298.  Keys that three or four entries read are better kept (N = 2^14, 24 rotations of four 389 / 415).
#define STREAMED_KEY_BYTES ((u64)208 << 20)
#define NONTEMPORAL 2    // of a buffer access

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

// ---- rows of 1024 coefficients, one wave each (convert_fp.hip, convert_int.hip) ----
#define ROW_LDS 1056     // 64-bit words per wave: 32 x 33, one pad word per 32
#define ROWS_NT 256

// Position of a limb -> its prime: the l limbs of q first, special limbs behind them.
__device__ __forceinline__ int prime_at(int pos, int l, int L) { return pos < l ? pos : pos + (L - l); }

// Byte offsets of the elements that sigma_g moves to 1024 row + 64 r + lane.  The exponent of index i is 2 bitrev(i) + 1,
// its product with g splits into a term of the lane (one multiplication) and a uniform term of (row, r); shifting both left
// by 31 - log2 N makes the 32-bit sum wrap modulo 2N, and reversing its bits gives the source index with the bit of the
// always-odd exponent above it.
struct Gather {
    uint32_t lane_term, shift, row, log_n;
};
__device__ __forceinline__ Gather make_gather(u64 g, uint32_t row, int lane, int log_n) {
    const uint32_t gs = (uint32_t)g << (31 - log_n);
    uint32_t lane_term = (2u * (__brev((uint32_t)lane) >> (32 - log_n)) + 1u) * gs;
    asm volatile("" : "+v"(lane_term));      // otherwise the sum of products below becomes a product per register again
    return Gather{lane_term, gs, row, (uint32_t)log_n};
}
__device__ __forceinline__ uint32_t gather_offset(const Gather& t, int r) {
    const uint32_t u = t.lane_term + 2u * (__brev(t.row * 1024u + (uint32_t)r * 64u) >> (32 - t.log_n)) * t.shift;
    return (__brev(u) << 3) - (8u << t.log_n);
}

// Wave-level tasks, ordered (limb, row, entry): the entries of a row share its twiddles (5 KB beside 8 KB of data) and, in
// the inner product, its key rows (16 KB a digit), so the four waves of a workgroup find them in the L1 and the workgroups
// of an XCD (round-robin by id, hence the contiguous range per XCD) in its L2.
__device__ __forceinline__ int row_task(int n_tasks) {
    const int n_blocks = (n_tasks + 3) >> 2, per = (n_blocks + 7) >> 3;
    const int blk = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if ((int)(blockIdx.x >> 3) >= per) return -1;
    const int task = blk * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    return task < n_tasks ? task : -1;
}

// ---- rows of 1024 coefficients, four waves each: calls with few rows (V = double, B = float; V = u64, B = int) ----
// A wave that keeps a row to itself works through eighty butterflies a lane one after the other and fetches its twiddles in
// batches between them; with fewer rows than the chip has SIMDs nothing covers either.  Here a thread holds four
// coefficients, two levels at a time, and everything it will need is on its way before the first level; only the exchange
// behind the first two levels crosses waves.
//   stage s, levels 2 s and 2 s + 1: registers 0 .. 3 of thread t are 2^p apart, p = 8 - 2 s (wide_element)
#define WIDE_NT 256
#define WIDE_SPLIT 256   // inner products: workgroups of one polynomial each, while there is a compute unit for every one
#define WIDE_LDS 1280    // 64-bit words per row: four words of padding per sixteen, so that a thread's four stay together
__device__ __forceinline__ uint32_t wide_at(uint32_t i) { return i + ((i >> 4) << 2); }
template <int S>
__device__ __forceinline__ uint32_t wide_element(uint32_t t, uint32_t r) {
    constexpr int p = 8 - 2 * S;
    return ((t >> p) << (p + 2)) | (r << p) | (t & ((1u << p) - 1));
}
// registers of stage FROM to registers of stage TO; the waves keep to their quarter of the row except between stages 0 and 1
template <int FROM, int TO, class V, class B>
__device__ __forceinline__ void wide_exchange(V (&v)[4], B (&m)[4], V* lds, uint32_t t) {
    B top = 0;
#pragma unroll
    for (int r = 0; r < 4; r++) {
        lds[wide_at(wide_element<FROM>(t, r))] = v[r];
        top = m[r] > top ? m[r] : top;
    }
    xchg_sync<FROM + TO != 1>();
#pragma unroll
    for (int r = 0; r < 4; r++) {
        v[r] = lds[wide_at(wide_element<TO>(t, r))];
        m[r] = top;
    }
    xchg_sync<true>();
}
// The ten levels, bounds m in and out; bfly(stage, x, y, bound of x, of y, k): butterfly by twiddle k of the stage, 0 of its
// first level, 1 and 2 of the groups of its second.  The row's LDS is free when the first of its threads comes here.  Either
// meets the workgroup's barrier once: its threads that transform no row meet it in wide_no_row instead.
// forward: coefficient 256 r + t -> 4 t + r
template <int S = 0, class V, class B, class F>
__device__ __forceinline__ void wide_forward_levels(V (&v)[4], B (&m)[4], V* lds, uint32_t t, F bfly) {
    constexpr std::integral_constant<int, S> s{};
    bfly(s, v[0], v[2], m[0], m[2], 0);
    bfly(s, v[1], v[3], m[1], m[3], 0);
    bfly(s, v[0], v[1], m[0], m[1], 1);
    bfly(s, v[2], v[3], m[2], m[3], 2);
    if constexpr (S < 4) {
        wide_exchange<S, S + 1>(v, m, lds, t);
        wide_forward_levels<S + 1>(v, m, lds, t, bfly);
    }
}
// inverse: coefficient 4 t + r -> 256 r + t
template <int S = 4, class V, class B, class F>
__device__ __forceinline__ void wide_inverse_levels(V (&v)[4], B (&m)[4], V* lds, uint32_t t, F bfly) {
    constexpr std::integral_constant<int, S> s{};
    bfly(s, v[0], v[1], m[0], m[1], 1);
    bfly(s, v[2], v[3], m[2], m[3], 2);
    bfly(s, v[0], v[2], m[0], m[2], 0);
    bfly(s, v[1], v[3], m[1], m[3], 0);
    if constexpr (S > 0) {
        wide_exchange<S, S - 1>(v, m, lds, t);
        wide_inverse_levels<S - 1>(v, m, lds, t, bfly);
    }
}
__device__ __forceinline__ void wide_no_row() { xchg_sync<false>(); }

// coefficients 4 t + r of a limb's row, read through sigma_g when galois != 0
template <int K3, class V>
__device__ __forceinline__ void wide_load(V (&v)[4], const void* limb, u64 galois, uint32_t row, uint32_t t) {
    if (galois) {
        const rsrc_t src = make_rsrc(limb, (uint32_t)8192 << K3);
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const uint32_t at = galois_src_fp(row * 1024u + 4u * t + (uint32_t)r, galois, 10 + K3) * 8u;
            if constexpr (std::is_same_v<V, double>) v[r] = bloadf(src, at, 0);
            else v[r] = bload(src, at, 0);
        }
    } else {
        const rsrc_t src = make_rsrc((const u64*)limb + row * 1024u, 8192u);
        bload2(src, t * 32u, 0, v[0], v[1]);
        bload2(src, t * 32u, 16, v[2], v[3]);
    }
}
template <class V>
__device__ __forceinline__ void wide_store(rsrc_t dst, uint32_t t, const V (&v)[4]) {      // 4 t + r
    bstore2(dst, t * 32u, 0, v[0], v[1]);
    bstore2(dst, t * 32u, 16, v[2], v[3]);
}
// workgroups are tasks, (limb, row, entry) as above: a contiguous range of them per XCD
__device__ __forceinline__ int wide_task(int n_tasks) {
    const int per = (n_tasks + 7) >> 3, task = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    return (int)(blockIdx.x >> 3) < per && task < n_tasks ? task : -1;
}
