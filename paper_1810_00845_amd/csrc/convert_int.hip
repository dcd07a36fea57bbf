// Transforms, base conversion and key inner product in 64-bit integers: every ring degree 2^10 .. 2^16 and primes up to
// 60 bits (contexts that convert_fp.hip does not cover), with the same division of work as there.  A coefficient index is
// (a : log2 N - 10)(b : 5)(c : 5); the levels on `a` are done per column, one lane per column and 2^(log2 N - 10) registers,
// the ten levels on b and c per row of 1024 neighbours, one wave each and 16 coefficients a lane.
//   key switch   rows (inverse) -> columns (inverse levels, conversion inputs to LDS, conversion, forward levels) -> rows
//                (forward levels, inner product with the key, inverse rows of the special limbs) -> columns (division by P)
//                -> rows (forward levels, difference, addend)
//   rescale      rows -> columns -> rows, the same with one source limb
//   transforms   columns -> rows, or rows -> columns
// Five launches where one launch per step and digit made 22 (N = 2^12, 3 limbs, one rotation: 153 -> 45 us, 29 with the
// rows shared by four waves), and levels in registers where every level was a pass through LDS (N = 2^15, 8 limbs of 58 bits, 16
// rotations: 685 -> 374 us, 332 with the inner products shared out over the XCDs).
//
// Arithmetic: a product with a constant w uses its companion floor(2^64 w / q); the quotient is formed without the product
// of the low halves and with the two middle ones truncated, so it is short by at most 3 and the product lies below 4 q
// for ANY 64-bit factor (13 instructions against 17 for the exact quotient; all of them issue at the same rate here).
// q < 2^60 leaves room for values below 16 q: bounds are counted at compile time (in units of q) and a conditional
// subtraction of 8 q is placed where a sum could exceed 16 q.  Products of two variables are summed over 30-bit halves in
// three 64-bit accumulators (four multiply-adds a term, no carries) and reduced once.
#include <cstdio>

#include "fp_device.hpp"
#include "modarith.hpp"

typedef const __attribute__((address_space(4))) u64* cu64_ptr;
__device__ __forceinline__ cu64_ptr as_constu(const u64* p) { return (cu64_ptr)(unsigned long long)p; }

#define CLOSE_WORDS 4    // per source limb: factor f and companion, f times the last inverse twiddle and companion
#define CONST_WORDS 6    // per prime: the same for f = N^-1, then WideMod
#define MASK30 0x3fffffffu

struct ModI { u64 q, r1; };      // r1 = floor(2^64 / q)
__device__ __forceinline__ ModI mod_int(const PrimeConst* primes, int prime) {
    return ModI{as_constu(&primes[prime].q)[0], as_constu(&primes[prime].q)[1]};
}

// (16-bit kernel arguments come through vector loads: without this every descriptor built from them took a loop over lanes)
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

struct Tw { u64 w, s; };

// a w mod q, below 4 q, for any a
__device__ __forceinline__ u64 approx_mulhi(u64 a, u64 s) {
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), s0 = (uint32_t)s, s1 = (uint32_t)(s >> 32);
    return (u64)a1 * s1 + ((u64)__umulhi(a1, s0) + (u64)__umulhi(a0, s1));
}
// low word of a product, opaque: the compiler would merge it with an addition into a 64-bit multiply-add and two moves
__device__ __forceinline__ uint32_t mul_lo(uint32_t a, uint32_t b) {
    uint32_t r = a * b;
    asm("" : "+v"(r));
    return r;
}
// x + a w - h q, the additions inside the multiply-adds (nq = -q modulo 2^64): a 64-bit subtraction costs a carry hazard
__device__ __forceinline__ u64 mad_sub(u64 x, u64 a, u64 w, u64 h, u64 nq) {
    const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32), w0 = (uint32_t)w, w1 = (uint32_t)(w >> 32);
    const uint32_t h0 = (uint32_t)h, h1 = (uint32_t)(h >> 32), n0 = (uint32_t)nq, n1 = (uint32_t)(nq >> 32);
    const u64 lo = (u64)h0 * n0 + ((u64)a0 * w0 + x);
    const uint32_t hi = (uint32_t)(lo >> 32) + (mul_lo(a0, w1) + mul_lo(a1, w0)) + (mul_lo(h0, n1) + mul_lo(h1, n0));
    return ((u64)hi << 32) | (uint32_t)lo;
}
__device__ __forceinline__ u64 mul4(u64 a, Tw t, u64 q) { return mad_sub(0, a, t.w, approx_mulhi(a, t.s), 0 - q); }
__device__ __forceinline__ u64 reduce4(u64 a, ModI q) { return mul4(a, Tw{1, q.r1}, q.q); }

__device__ __forceinline__ u64 sub_if(u64 x, u64 k) {          // x >= k ? x - k : x, for x < 2 k <= 2^64
    u64 d;                                                     // (the compiler makes a subtraction and a 64-bit comparison of it)
    asm("v_lshl_add_u64 %0, %1, 0, %2" : "=v"(d) : "v"(x), "s"(0 - k));
    return (int32_t)(d >> 32) < 0 ? x : d;
}
// x below m q (m <= 16) -> below the returned multiple, at most `cap`
__device__ __forceinline__ void cap_to(u64& x, int& m, int cap, u64 q) {
    if (m > 8 && cap < 16) { x = sub_if(x, q << 3); m = 8; }
    if (m > 4 && cap < 8) { x = sub_if(x, q << 2); m = 4; }
    if (m > 2 && cap < 4) { x = sub_if(x, q << 1); m = 2; }
    if (m > 1 && cap < 2) { x = sub_if(x, q); m = 1; }
}
__device__ __forceinline__ u64 canonical(u64 x, int m, u64 q) { cap_to(x, m, 1, q); return x; }

// forward butterfly: (x, y) -> (x + w y, x - w y)
__device__ __forceinline__ void fwd_bfly(u64& x, u64& y, int& bx, int& by, Tw w, u64 q) {
    if (bx > 12) cap_to(x, bx, 8, q);
    const u64 t = mul4(y, w, q);
    y = x + (q << 2) - t;
    x = x + t;
    bx = by = bx + 4;
}
// inverse butterfly: (x, y) -> (x + y, (x - y) w)
__device__ __forceinline__ void inv_bfly(u64& x, u64& y, int& bx, int& by, Tw w, u64 q) {
    cap_to(x, bx, 8, q);
    cap_to(y, by, 8, q);
    const u64 d = x + (by > 4 ? q << 3 : q << 2) - y;
    x = x + y;
    bx = bx + by;
    y = mul4(d, w, q);
    by = 4;
}

__device__ __forceinline__ void swap_halves(u64& x, u64& y) {
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    x = ((u64)hi[0] << 32) | lo[0];
    y = ((u64)hi[1] << 32) | lo[1];
}

// Five levels on a five-bit field, elements and twiddles as in convert_fp.hip: register r of half h holds element 2 r + h
// before and 4 (r >> 1) + 2 h + (r & 1) after the forward levels; t[g]: twiddles of level J < 4, last[k]: level 4, group
// 2 k + h.
template <int J>
__device__ __forceinline__ void fwd_level(u64 (&v)[16], int (&m)[16], const Tw (&t)[1 << J], u64 q) {
    constexpr int half = 3 - J;
#pragma unroll
    for (int g = 0; g < (1 << J); g++)
#pragma unroll
        for (int lo = 0; lo < (1 << half); lo++) {
            const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
            fwd_bfly(v[r0], v[r1], m[r0], m[r1], t[g], q);
        }
}
template <int J>
__device__ __forceinline__ void inv_level(u64 (&v)[16], int (&m)[16], const Tw (&t)[1 << J], u64 q) {
    constexpr int half = 3 - J;
#pragma unroll
    for (int g = 0; g < (1 << J); g++)
#pragma unroll
        for (int lo = 0; lo < (1 << half); lo++) {
            const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
            inv_bfly(v[r0], v[r1], m[r0], m[r1], t[g], q);
        }
}
__device__ __forceinline__ void fwd_last(u64 (&v)[16], int (&m)[16], const Tw (&t)[8], u64 q) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
        swap_halves(v[2 * k], v[2 * k + 1]);
        m[2 * k] = m[2 * k + 1] = m[2 * k] > m[2 * k + 1] ? m[2 * k] : m[2 * k + 1];
        fwd_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], t[k], q);
    }
}
__device__ __forceinline__ void inv_last(u64 (&v)[16], int (&m)[16], const Tw (&t)[8], u64 q) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
        inv_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], t[k], q);
        swap_halves(v[2 * k], v[2 * k + 1]);
        m[2 * k] = m[2 * k + 1] = m[2 * k] > m[2 * k + 1] ? m[2 * k] : m[2 * k + 1];
    }
}

// one bound for all registers, at most cap (values change lanes and registers in an exchange)
__device__ __forceinline__ void cap_bounds(u64 (&v)[16], int (&m)[16], int cap, u64 q) {
    int top = 0;
#pragma unroll
    for (int r = 0; r < 16; r++) {
        cap_to(v[r], m[r], cap, q);
        top = m[r] > top ? m[r] : top;
    }
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = top;
}

// Twiddles of a row straight from the tables in bit-reversed order: level k of the transform, group i at entry 2^k + i.
template <int K3>
struct RowTables {
    const u64 *w, *s;
    rsrc_t wr, sr;
    uint32_t row, lane;
    __device__ __forceinline__ RowTables(const u64* tw, const u64* tw_sh, int prime, uint32_t row_, int lane_) : row(row_), lane((uint32_t)lane_) {
        constexpr u64 n = (u64)1 << (10 + K3);
        w = tw + (u64)prime * n;
        s = tw_sh + (u64)prime * n;
        wr = make_rsrc(w, (uint32_t)n * 8u);
        sr = make_rsrc(s, (uint32_t)n * 8u);
    }
    __device__ __forceinline__ Tw at(uint32_t i) const { return Tw{bload(wr, i * 8u, 0), bload(sr, i * 8u, 0)}; }
    template <int J> __device__ __forceinline__ void b(Tw (&t)[1 << J]) const {          // uniform: scalar loads
#pragma unroll
        for (int g = 0; g < (1 << J); g++) {
            const uint32_t i = (((1u << K3) + row) << J) + (uint32_t)g;
            t[g] = Tw{as_constu(w)[i], as_constu(s)[i]};
        }
    }
    __device__ __forceinline__ void b_last(Tw (&t)[8]) const {
#pragma unroll
        for (int k = 0; k < 8; k++) t[k] = at((((1u << K3) + row) << 4) + 2u * k + (lane >> 5));
    }
    template <int J> __device__ __forceinline__ void c(Tw (&t)[1 << J]) const {
#pragma unroll
        for (int g = 0; g < (1 << J); g++) t[g] = at((node() << J) + (uint32_t)g);
    }
    __device__ __forceinline__ void c_last(Tw (&t)[8]) const {
#pragma unroll
        for (int k = 0; k < 8; k++) t[k] = at((node() << 4) + 2u * k + (lane >> 5));
    }
    __device__ __forceinline__ uint32_t node() const { return 32u * ((1u << K3) + row) + (lane & 31u); }
};

// The ten levels of a row; register r of lane i is coefficient 64 r + i before and after.
template <int K3, class PUT>
__device__ __forceinline__ void row_forward(u64 (&v)[16], int (&m)[16], const RowTables<K3>& w, u64* lds, int lane, u64 q, int cap, PUT put) {
    const int h = lane >> 5, s = lane & 31;
    Tw t0[1], t1[2], t2[4], t3[8], last[8];
    w.template b<0>(t0); w.template b<1>(t1); w.template b<2>(t2); w.template b<3>(t3);
    fwd_level<0>(v, m, t0, q); fwd_level<1>(v, m, t1, q); fwd_level<2>(v, m, t2, q); fwd_level<3>(v, m, t3, q);
    w.b_last(last);
    fwd_last(v, m, last, q);
    cap_bounds(v, m, 16, q);
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[(2 * h + (r >> 1) * 4 + (r & 1)) * 33 + s] = v[r];
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[s * 33 + h + 2 * r];
    w.template c<0>(t0); w.template c<1>(t1); w.template c<2>(t2);
    fwd_level<0>(v, m, t0, q); fwd_level<1>(v, m, t1, q); fwd_level<2>(v, m, t2, q);
    w.template c<3>(t3);
    fwd_level<3>(v, m, t3, q);
    w.c_last(last);
    fwd_last(v, m, last, q);
    cap_bounds(v, m, cap, q);
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[s * 33 + 2 * h + (r >> 1) * 4 + (r & 1)] = put(v[r]);
    xchg_sync<true>();
}
template <int K3>
__device__ __forceinline__ void row_forward(u64 (&v)[16], int (&m)[16], const RowTables<K3>& w, u64* lds, int lane, u64 q, int cap) {
    row_forward(v, m, w, lds, lane, q, cap, [](u64 x) { return x; });
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[66 * r + lane + (lane >> 5)];
}
// the row lies in LDS already, coefficient i at i + i / 32, below m q
template <int K3>
__device__ __forceinline__ void row_inverse_lds(u64 (&v)[16], int (&m)[16], const RowTables<K3>& w, u64* lds, int lane, u64 q) {
    const int h = lane >> 5, s = lane & 31;
    Tw t0[1], t1[2], t2[4], t3[8], last[8];
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[s * 33 + 2 * h + (r >> 1) * 4 + (r & 1)];
    w.c_last(last);
    inv_last(v, m, last, q);
    w.template c<3>(t3);
    inv_level<3>(v, m, t3, q);
    w.template c<2>(t2); w.template c<1>(t1); w.template c<0>(t0);
    inv_level<2>(v, m, t2, q); inv_level<1>(v, m, t1, q); inv_level<0>(v, m, t0, q);
    cap_bounds(v, m, 16, q);
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[s * 33 + h + 2 * r] = v[r];
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[(2 * h + (r >> 1) * 4 + (r & 1)) * 33 + s];
    w.b_last(last);
    inv_last(v, m, last, q);
    w.template b<3>(t3); w.template b<2>(t2); w.template b<1>(t1); w.template b<0>(t0);
    inv_level<3>(v, m, t3, q); inv_level<2>(v, m, t2, q); inv_level<1>(v, m, t1, q); inv_level<0>(v, m, t0, q);
    cap_bounds(v, m, 8, q);
}
template <int K3>
__device__ __forceinline__ void row_inverse(u64 (&v)[16], int (&m)[16], const RowTables<K3>& w, u64* lds, int lane, u64 q) {
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[66 * r + lane + (lane >> 5)] = v[r];
    xchg_sync<true>();
    row_inverse_lds(v, m, w, lds, lane, q);
}

// the row's 1024 words of a limb, read through sigma_g when galois != 0
template <int K3>
__device__ __forceinline__ void load_row(u64 (&v)[16], const u64* limb, u64 galois, uint32_t row, int lane) {
    if (galois) {
        const rsrc_t src = make_rsrc(limb, (uint32_t)8192 << K3);
        const Gather t = make_gather(galois, row, lane, 10 + K3);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = bload(src, gather_offset(t, r), 0);
    } else {
        const rsrc_t src = make_rsrc(limb + row * 1024u, 8192u);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = bload(src, (uint32_t)lane * 8u, (uint32_t)r * 512u);
    }
}

// ---- sums of products over 30-bit halves ----
__device__ __forceinline__ u64 split30(u64 x) { return ((x >> 30) << 32) | ((uint32_t)x & MASK30); }
struct Acc3 { u64 lo, mid, hi; };
__device__ __forceinline__ void acc3_mad(Acc3& a, u64 x, u64 y) {
    const uint32_t x0 = (uint32_t)x, x1 = (uint32_t)(x >> 32), y0 = (uint32_t)y, y1 = (uint32_t)(y >> 32);
    a.lo += (u64)x0 * y0;
    a.mid += (u64)x0 * y1;
    a.mid += (u64)x1 * y0;
    a.hi += (u64)x1 * y1;
}
// The sum T below 2^63 q -> T mod q, below 6 q: the quotient is (T >> k - 1) floor(2^(63 + k) / q) >> 64 with k bits of q,
// short by the three of mul4, one for the bits shifted out and one for the truncated reciprocal.
struct WideMod { u64 recip; uint32_t k1; };     // floor(2^(63 + k) / q), k - 1
__device__ __forceinline__ u64 acc3_reduce(Acc3 a, WideMod w, u64 q) {
    a.mid += a.lo >> 30;
    a.hi += a.mid >> 30;
    const u64 low = ((a.mid & MASK30) << 30) | (a.lo & MASK30);
    const u64 t = (a.hi << (60 - w.k1)) | (low >> w.k1);
    const u64 h = approx_mulhi(t, w.recip), nq = 0 - q;
    const uint32_t h0 = (uint32_t)h, h1 = (uint32_t)(h >> 32), n0 = (uint32_t)nq, n1 = (uint32_t)(nq >> 32);
    const u64 lo = (u64)h0 * n0 + (low + (a.hi << 60));
    return ((u64)((uint32_t)(lo >> 32) + (mul_lo(h0, n1) + mul_lo(h1, n0))) << 32) | (uint32_t)lo;
}
__device__ __forceinline__ WideMod wide_mod(const u64* consts, int prime) {
    return WideMod{as_constu(consts)[(u64)prime * CONST_WORDS + 4], (uint32_t)as_constu(consts)[(u64)prime * CONST_WORDS + 5]};
}
__device__ __forceinline__ Tw table_tw(const u64* t, u64 i) { return Tw{as_constu(t)[i], as_constu(t)[i + 1]}; }

// ---------------------------------------------------------------------------
// rows
// ---------------------------------------------------------------------------
template <int K3>
__device__ __forceinline__ void rows_inverse(const IntArgs& a, const IntTasks& tk, int n_tasks, u64* lds_all) {
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    const uint32_t unit = uniform((uint32_t)task / a.n_entries), row = unit & ((1u << K3) - 1), e = unit >> K3;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const int prime = uniform(tk.prime[e]), pos = uniform(tk.pos[e]);
    const ModI q = mod_int(a.primes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    u64 v[16];
    int m[16];
    load_row<K3>(v, a.in + b * a.in_bs + (u64)(pos + a.in_pos_shift) * n, a.galois, row, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = 1;
    row_inverse<K3>(v, m, RowTables<K3>(a.itw, a.itw_sh, prime, row, lane), lds_all + (threadIdx.x >> 6) * ROW_LDS, lane, q.q);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)pos * n + (uint32_t)uniform(row) * 1024u, 8192u);
    if (K3 == 0 && a.whole) {            // no columns behind
        const Tw f = table_tw(a.consts, (u64)prime * CONST_WORDS);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = canonical(mul4(v[r], f, q.q), 4, q.q);
    }
#pragma unroll
    for (int r = 0; r < 16; r++) bstore(dst, (uint32_t)lane * 8u, (uint32_t)r * 512u, v[r]);
}

template <int K3>
__device__ __forceinline__ void rows_forward(const IntArgs& a, const IntTasks& tk, int n_tasks, u64* lds_all) {
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    const uint32_t unit = uniform((uint32_t)task / a.n_entries), row = unit & ((1u << K3) - 1), e = unit >> K3;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const int prime = uniform(tk.prime[e]), pos = uniform(tk.pos[e]);
    const ModI q = mod_int(a.primes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)pos * n + row * 1024u, 8192u);
    // without levels on `a` in front the polynomial is where the caller left it
    const bool direct = K3 == 0 && a.in && !a.coeffs;
    const rsrc_t src = direct ? make_rsrc(a.in + b * a.in_bs + (u64)(pos + a.in_pos_shift) * n, 8192u) : dst;
    u64 v[16];
    int m[16];
#pragma unroll
    for (int r = 0; r < 16; r++) { v[r] = bload(src, (uint32_t)lane * 8u, (uint32_t)r * 512u); m[r] = 16; }
    row_forward<K3>(v, m, RowTables<K3>(a.tw, a.tw_sh, prime, row, lane), lds_all + (threadIdx.x >> 6) * ROW_LDS, lane, q.q, 16);
#pragma unroll
    for (int r = 0; r < 16; r++) bstore(dst, (uint32_t)lane * 8u, (uint32_t)r * 512u, canonical(v[r], 16, q.q));
}

// behind a division's columns: out = (acc - transform) * factor (+ addend)
template <int K3>
__device__ __forceinline__ void rows_divide(const IntArgs& a, int n_tasks, u64* lds_all) {
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    const uint32_t unit = uniform((uint32_t)task / a.n_entries), row = unit & ((1u << K3) - 1), e = unit >> K3;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const ModI q = mod_int(a.primes, (int)e);
    constexpr u64 n = (u64)1 << (10 + K3);
    const uint32_t lane8 = (uint32_t)lane * 8u;
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)e * n + row * 1024u, 8192u);
    const rsrc_t acc = make_rsrc(a.acc + b * a.acc_bs + (u64)e * n + row * 1024u, 8192u);
    u64 v[16], t[16];
    int m[16];
#pragma unroll
    for (int r = 0; r < 16; r++) { v[r] = bload(dst, lane8, (uint32_t)r * 512u); m[r] = 16; }
    row_forward<K3>(v, m, RowTables<K3>(a.tw, a.tw_sh, (int)e, row, lane), lds_all + (threadIdx.x >> 6) * ROW_LDS, lane, q.q, 8);
    const Tw f = Tw{as_constu(a.factor)[e], as_constu(a.factor_sh)[e]};
#pragma unroll
    for (int r = 0; r < 16; r++) t[r] = bload(acc, lane8, (uint32_t)r * 512u);
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = mul4(t[r] + (q.q << 3) - v[r], f, q.q);           // acc is below 8 q
    if (a.add && (int)(b % a.add_div) < a.add_polys) {
        load_row<K3>(t, a.add + (b / a.add_div) * a.add_bs + (b % a.add_div) * a.add_ps + (u64)e * n, a.add_galois, row, lane);
#pragma unroll
        for (int r = 0; r < 16; r++) bstore(dst, lane8, (uint32_t)r * 512u, canonical(v[r] + t[r], 5, q.q));
    } else {
#pragma unroll
        for (int r = 0; r < 16; r++) bstore(dst, lane8, (uint32_t)r * 512u, canonical(v[r], 4, q.q));
    }
}

// Behind the columns of a key switch's digits.  One workgroup per (limb x, row, entry).  First a wave per digit, up to
// INNER_CHUNK of them: forward levels, or for the limb's own digit the input itself, read through sigma_g; the rows are left in
// LDS in 30-bit halves.  Then the waves share out the coefficients, groups of INNER_GROUP registers: sums of the digits
// times both polynomials of the key.  Limbs of q leave as accumulators (below 8 q); those of special limbs replace the first
// two rows in LDS and two waves take them through the inverse levels of the row, which the division by P starts with.
//
// Workgroups go round the XCDs by number.  An XCD takes every eighth row (or, with fewer than eight rows, its share of the
// limbs of one) and works through the limbs of its rows, the special ones first: they take longest, and with the limbs
// handed out in order three XCDs had all of them (16 rotations at N = 2^15, 8 limbs of 58 bits: 166 us a launch, 127 so; 64 rotations at
// N = 2^13: 41 -> 31).  The entries of a row and limb follow one another: they share its key rows.
struct InnerTask { int x; uint32_t row; u64 b; };
__host__ __device__ constexpr uint32_t inner_rows(int k3) { return k3 < 3 ? 1u : 1u << (k3 - 3); }             // of an XCD
__host__ __device__ constexpr uint32_t inner_parts(int k3) { return k3 < 3 ? 8u >> k3 : 1u; }                   // XCDs to a row
template <int K3>
__device__ __forceinline__ InnerTask inner_task(const IntArgs& a) {
    const uint32_t xcd = blockIdx.x & 7, unit = (uint32_t)uniform((int)((blockIdx.x >> 3) / a.n_entries));
    const u64 b = (blockIdx.x >> 3) - unit * a.n_entries;
    constexpr uint32_t ROWS = inner_rows(K3), PARTS = inner_parts(K3);
    const uint32_t row = K3 < 3 ? xcd / PARTS : xcd + 8 * (unit % ROWS);
    return InnerTask{a.ext_limbs - 1 - (int)(unit / ROWS * PARTS + (K3 < 3 ? xcd % PARTS : 0)), row, b};
}
#define INNER_CHUNK 4    // four terms below 2 q times q keep the middle accumulator below 2^64 and the sum below 2^63 q
#define INNER_GROUP 2    // times two polynomials: 24 registers of accumulators
template <int K3>
__device__ __forceinline__ void rows_inner(const IntArgs& a, u64* lds) {
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    const InnerTask it = inner_task<K3>(a);
    if (it.x < 0) return;
    const uint32_t row = it.row;
    const u64 b = it.b;
    const int x = it.x;
    const int prime = prime_at(x, a.l, a.L);
    const ModI q = mod_int(a.primes, prime);
    const WideMod wide = wide_mod(a.consts, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    const uint32_t lane8 = (uint32_t)lane * 8u;
    const bool special = x >= a.l;
    const u64 poly_words = (special ? (u64)(a.ext_limbs - a.l) : (u64)a.l) * n;
    u64* to = special ? a.down + b * 2 * poly_words + (u64)(x - a.l) * n : a.sums + b * 2 * poly_words + (u64)x * n;
    const rsrc_t dst = make_rsrc(to + row * 1024u, (uint32_t)(poly_words * 8u) + 8192u);
    for (int d0 = 0; d0 < a.n_digits; d0 += INNER_CHUNK) {
        const int d1 = min(d0 + INNER_CHUNK, a.n_digits);
        if (d0) __syncthreads();                                // the rows of the chunk before are done with
        for (int d = d0 + wave; d < d1; d += waves) {
            u64* slot = lds + (d - d0) * ROW_LDS;
            u64 v[16];
            if (x >= d * a.alpha && x < min((d + 1) * a.alpha, a.l)) {
                load_row<K3>(v, a.in + b * a.in_bs + (u64)x * n, a.galois, row, lane);
#pragma unroll
                for (int r = 0; r < 16; r++) slot[66 * r + lane + h] = split30(v[r]);
            } else {
                const rsrc_t src = make_rsrc(a.ext + b * a.ext_bs + (u64)(d * a.ext_limbs + x) * n + row * 1024u, 8192u);
                int m[16];
#pragma unroll
                for (int r = 0; r < 16; r++) { v[r] = bload(src, lane8, (uint32_t)r * 512u); m[r] = 16; }
                row_forward(v, m, RowTables<K3>(a.tw, a.tw_sh, prime, row, lane), slot, lane, q.q, 2, [](u64 y) { return split30(y); });
            }
        }
        __syncthreads();
        const u64* key_p = a.key + ((u64)d0 * 2 * a.total + prime) * n + row * 1024u;
        for (int r0 = wave * INNER_GROUP; r0 < 16; r0 += waves * INNER_GROUP) {
            Acc3 acc[2][INNER_GROUP];
            const uint32_t r8 = (uint32_t)r0 * 512u;
            u64* slot = lds + 66 * r0 + lane + h;
#pragma unroll
            for (int r = 0; r < INNER_GROUP; r++) acc[0][r] = acc[1][r] = Acc3{0, 0, 0};
#pragma unroll 2
            for (int d = 0; d < d1 - d0; d++) {
                u64 k[2][INNER_GROUP];
#pragma unroll
                for (int p = 0; p < 2; p++) {
                    const rsrc_t key = make_rsrc(key_p + (u64)(2 * d + p) * a.total * n, 8192u);
#pragma unroll
                    for (int r = 0; r < INNER_GROUP; r++) k[p][r] = bload(key, lane8, r8 + (uint32_t)r * 512u);
                }
#pragma unroll
                for (int r = 0; r < INNER_GROUP; r++) {
                    const u64 e = slot[d * ROW_LDS + 66 * r];
                    acc3_mad(acc[0][r], e, split30(k[0][r]));
                    acc3_mad(acc[1][r], e, split30(k[1][r]));
                }
            }
#pragma unroll
            for (int p = 0; p < 2; p++) {
#pragma unroll
                for (int r = 0; r < INNER_GROUP; r++) {
                    const uint32_t off = (uint32_t)(p * poly_words * 8u) + r8 + (uint32_t)r * 512u;
                    u64 s = acc3_reduce(acc[p][r], wide, q.q);
                    if (d0) s = sub_if(s + bload(dst, lane8, off), q.q << 3);     // sums of earlier chunks wait where the result goes
                    if (special && d1 == a.n_digits) slot[p * ROW_LDS + 66 * r] = s;
                    else bstore(dst, lane8, off, s);
                }
            }
        }
    }
    if (!special) return;
    __syncthreads();
    if (wave >= 2) return;
    u64 v[16];
    int m[16];
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = 8;
    row_inverse_lds(v, m, RowTables<K3>(a.itw, a.itw_sh, prime, row, lane), lds + wave * ROW_LDS, lane, q.q);
#pragma unroll
    for (int r = 0; r < 16; r++) bstore(dst, lane8, (uint32_t)(wave * poly_words * 8u) + (uint32_t)r * 512u, v[r]);
}

// ---------------------------------------------------------------------------
// rows by four waves each: calls with few rows
// ---------------------------------------------------------------------------
struct WideTwiddles { Tw w[5][3]; };     // per stage: level 2 s, then the two groups of level 2 s + 1
template <int K3>
__device__ __forceinline__ void wide_twiddles(WideTwiddles& w, const u64* tw, const u64* tw_sh, int prime, uint32_t row, uint32_t t) {
    constexpr u64 n = (u64)1 << (10 + K3);
    const rsrc_t wr = make_rsrc(tw + (u64)prime * n, (uint32_t)n * 8u), sr = make_rsrc(tw_sh + (u64)prime * n, (uint32_t)n * 8u);
#pragma unroll
    for (int s = 0; s < 5; s++) {
        const uint32_t node = (((1u << K3) + row) << (2 * s)) + (t >> (8 - 2 * s));
        w.w[s][0] = Tw{bload(wr, node * 8u, 0), bload(sr, node * 8u, 0)};
        bload2(wr, node * 16u, 0, w.w[s][1].w, w.w[s][2].w);
        bload2(sr, node * 16u, 0, w.w[s][1].s, w.w[s][2].s);
    }
}
// out: below cap q
__device__ __forceinline__ void wide_forward(u64 (&v)[4], int (&m)[4], const WideTwiddles& w, u64* lds, uint32_t t, u64 q, int cap) {
    wide_forward_levels(v, m, lds, t, [&](auto s, u64& x, u64& y, int& bx, int& by, int k) { fwd_bfly(x, y, bx, by, w.w[s][k], q); });
#pragma unroll
    for (int r = 0; r < 4; r++) cap_to(v[r], m[r], cap, q);
}
// out: below 8 q
__device__ __forceinline__ void wide_inverse(u64 (&v)[4], int (&m)[4], const WideTwiddles& w, u64* lds, uint32_t t, u64 q) {
    wide_inverse_levels(v, m, lds, t, [&](auto s, u64& x, u64& y, int& bx, int& by, int k) { inv_bfly(x, y, bx, by, w.w[s][k], q); });
#pragma unroll
    for (int r = 0; r < 4; r++) cap_to(v[r], m[r], 8, q);
}

template <int K3>
__device__ __forceinline__ void wide_rows_inverse(const IntArgs& a, const IntTasks& tk, int task, u64* lds) {
    const uint32_t t = threadIdx.x, unit = uniform((uint32_t)task / a.n_entries), row = unit & ((1u << K3) - 1), e = unit >> K3;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const int prime = uniform(tk.prime[e]), pos = uniform(tk.pos[e]);
    const u64 q = mod_int(a.primes, prime).q;
    constexpr u64 n = (u64)1 << (10 + K3);
    u64 v[4];
    int m[4] = {1, 1, 1, 1};
    WideTwiddles w;
    wide_load<K3>(v, a.in + b * a.in_bs + (u64)(pos + a.in_pos_shift) * n, a.galois, row, t);
    wide_twiddles<K3>(w, a.itw, a.itw_sh, prime, row, t);
    wide_inverse(v, m, w, lds, t, q);
    if (K3 == 0 && a.whole) {            // no columns behind
        const Tw f = table_tw(a.consts, (u64)prime * CONST_WORDS);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = canonical(mul4(v[r], f, q), 4, q);
    }
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)pos * n + row * 1024u, 8192u);
#pragma unroll
    for (int r = 0; r < 4; r++) bstore(dst, t * 8u, (uint32_t)r * 2048u, v[r]);
}

template <int K3>
__device__ __forceinline__ void wide_rows_divide(const IntArgs& a, int task, u64* lds) {
    const uint32_t t = threadIdx.x, unit = uniform((uint32_t)task / a.n_entries), row = unit & ((1u << K3) - 1), e = unit >> K3;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const u64 q = mod_int(a.primes, (int)e).q;
    constexpr u64 n = (u64)1 << (10 + K3);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)e * n + row * 1024u, 8192u);
    const bool with_add = a.add && (int)(b % a.add_div) < a.add_polys;
    u64 v[4], acc[4], add[4] = {};
    int m[4] = {16, 16, 16, 16};
    WideTwiddles w;
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = bload(dst, t * 8u, (uint32_t)r * 2048u);
    wide_twiddles<K3>(w, a.tw, a.tw_sh, (int)e, row, t);
    wide_load<K3>(acc, a.acc + b * a.acc_bs + (u64)e * n, 0, row, t);
    if (with_add)
        wide_load<K3>(add, a.add + (b / a.add_div) * a.add_bs + (b % a.add_div) * a.add_ps + (u64)e * n, a.add_galois, row, t);
    const Tw f = Tw{as_constu(a.factor)[e], as_constu(a.factor_sh)[e]};
    wide_forward(v, m, w, lds, t, q, 8);
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = canonical(mul4(acc[r] + (q << 3) - v[r], f, q) + add[r], 5, q);     // acc is below 8 q
    wide_store(dst, t, v);
}

// A workgroup per (limb x, row, entry), four waves per digit (two digits at least, INNER_CHUNK at most: the caller's rule).  Each
// four leave their digit's row in LDS in 30-bit halves; then the first eight waves form the sums of a polynomial each, and
// take those of a special limb through the inverse levels.  split: a workgroup per polynomial too, as in convert_fp.hip.
template <int K3>
__device__ __forceinline__ void wide_rows_inner(const IntArgs& a, int task, u64* lds) {
    const uint32_t t = threadIdx.x & (WIDE_NT - 1);
    const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WIDE_NT));
    const uint32_t entry = (uint32_t)task >> a.split, unit = uniform(entry / a.n_entries), row = unit & ((1u << K3) - 1);
    const u64 b = entry - unit * a.n_entries;
    const int summer = a.n_digits < INNER_CHUNK ? a.n_digits : 0, poly = a.split ? task & 1 : part;
    const int x = a.ext_limbs - 1 - (int)(unit >> K3);
    const int prime = prime_at(x, a.l, a.L);
    const u64 q = mod_int(a.primes, prime).q;
    const WideMod wide = wide_mod(a.consts, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    const bool special = x >= a.l, sums = a.split ? part == summer : part < 2;
    u64 v[4], k[INNER_CHUNK][4];
    int m[4] = {16, 16, 16, 16};
    WideTwiddles w;
    u64* slot = lds + part * WIDE_LDS;
    const bool mine = part < a.n_digits, own = mine && x >= part * a.alpha && x < min((part + 1) * a.alpha, a.l);
    if (own) {
        wide_load<K3>(v, a.in + b * a.in_bs + (u64)x * n, a.galois, row, t);
    } else if (mine) {
        const rsrc_t src = make_rsrc(a.ext + b * a.ext_bs + (u64)(part * a.ext_limbs + x) * n + row * 1024u, 8192u);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = bload(src, t * 8u, (uint32_t)r * 2048u);
        wide_twiddles<K3>(w, a.tw, a.tw_sh, prime, row, t);
    }
    const bool waits = sums && !mine;                            // has no digit
    if (waits && special) wide_twiddles<K3>(w, a.itw, a.itw_sh, prime, row, t);
    if (sums) {
#pragma unroll
        for (int d = 0; d < INNER_CHUNK; d++)
            if (d < a.n_digits) wide_load<K3>(k[d], a.key + ((u64)(2 * d + poly) * a.total + prime) * n, 0, row, t);
    }
    if (mine && !own) wide_forward(v, m, w, slot, t, q, 2);
    else wide_no_row();
    if (mine) {
#pragma unroll
        for (int r = 0; r < 4; r++) slot[wide_at(4 * t + r)] = split30(v[r]);
    }
    if (sums && special && !waits) wide_twiddles<K3>(w, a.itw, a.itw_sh, prime, row, t);   // on their way while the sums are formed
    __syncthreads();
    if (sums) {
#pragma unroll
        for (int r = 0; r < 4; r++) {
            Acc3 acc = {0, 0, 0};
#pragma unroll
            for (int d = 0; d < INNER_CHUNK; d++)
                if (d < a.n_digits) acc3_mad(acc, lds[d * WIDE_LDS + wide_at(4 * t + r)], split30(k[d][r]));
            v[r] = acc3_reduce(acc, wide, q);
            m[r] = 8;
        }
        if (!special) {
            const rsrc_t dst = make_rsrc(a.sums + ((b * 2 + poly) * a.l + x) * n + row * 1024u, 8192u);
            wide_store(dst, t, v);
        }
    }
    if (!special) return;
    __syncthreads();                                            // everyone has read the digits
    if (!sums) {
        wide_no_row();
        return;
    }
    wide_inverse(v, m, w, slot, t, q);
    const rsrc_t dst = make_rsrc(a.down + ((b * 2 + poly) * (u64)(a.ext_limbs - a.l) + (u64)(x - a.l)) * n + row * 1024u, 8192u);
#pragma unroll
    for (int r = 0; r < 4; r++) bstore(dst, t * 8u, (uint32_t)r * 2048u, v[r]);
}

// ---------------------------------------------------------------------------
// columns
// ---------------------------------------------------------------------------
// A lane holds NR coefficients of its column.  From 32 rows on a column is shared by the two halves of the wave, as a row's
// fields are: half the registers, and the level on the lowest bit of `a` behind an exchange.
template <int RB>
struct Col {
    static constexpr bool SHARED = RB >= 5;
    static constexpr int LEVELS = SHARED ? RB - 1 : RB;      // levels inside a lane
    static constexpr int NR = 1 << LEVELS;
    static constexpr int WIDTH = SHARED ? 32 : 64, TILES = 1024 / WIDTH;
};
// byte offset of register r's row before the forward / after the inverse levels (FIRST) and on the other side; of the lane
template <int RB, bool FIRST>
__device__ __forceinline__ uint32_t column_row(int r) { return (uint32_t)(!Col<RB>::SHARED ? r : FIRST ? 2 * r : (r >> 1) * 4 + (r & 1)) * 8192u; }
template <int RB, bool FIRST>
__device__ __forceinline__ uint32_t column_lane(int tile, int lane) {
    return (uint32_t)(!Col<RB>::SHARED ? tile * 64 + lane : tile * 32 + (lane & 31) + (lane >> 5) * (FIRST ? 1024 : 2048)) * 8u;
}
// a column's twiddles: uniform ones, and those of the exchanged level
template <int RB>
struct ColTables {
    const u64 *w, *s;
    rsrc_t wr, sr;
    uint32_t half8;
    __device__ __forceinline__ ColTables(const u64* tw, const u64* tw_sh, int prime, int lane) {
        constexpr u64 n = (u64)1 << (10 + RB);
        w = tw + (u64)prime * n;
        s = tw_sh + (u64)prime * n;
        wr = make_rsrc(w, 8u << RB);
        sr = make_rsrc(s, 8u << RB);
        half8 = (uint32_t)(lane >> 5) * 8u;
    }
    __device__ __forceinline__ Tw at(int i) const { return Tw{as_constu(w)[i], as_constu(s)[i]}; }
    __device__ __forceinline__ Tw last(int k) const {
        const uint32_t o = (uint32_t)((1 << Col<RB>::LEVELS) + 2 * k) * 8u;
        return Tw{bload(wr, half8, o), bload(sr, half8, o)};
    }
};

// inverse levels on `a` of values below 8 q, the last one with the factor folded in (cl: CLOSE_WORDS words): canonical
template <int RB>
__device__ __forceinline__ void inv_columns(u64 (&v)[Col<RB>::NR], const ColTables<RB>& t, const u64* cl, u64 q) {
    constexpr int NR = Col<RB>::NR, LV = Col<RB>::LEVELS;
    const Tw f = table_tw(cl, 0);
    if constexpr (RB == 0) {
        v[0] = canonical(mul4(v[0], f, q), 4, q);
    } else {
        int m[NR];
#pragma unroll
        for (int r = 0; r < NR; r++) m[r] = 8;
        if constexpr (Col<RB>::SHARED) {
#pragma unroll
            for (int k = 0; k < NR / 2; k++) {
                inv_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], t.last(k), q);
                swap_halves(v[2 * k], v[2 * k + 1]);
                m[2 * k] = m[2 * k + 1] = m[2 * k] > m[2 * k + 1] ? m[2 * k] : m[2 * k + 1];
            }
        }
#pragma unroll
        for (int j = LV - 1; j >= 1; j--) {
            const int half = LV - 1 - j;
#pragma unroll
            for (int g = 0; g < (1 << j); g++) {
                const Tw w = t.at((1 << j) + g);
#pragma unroll
                for (int lo = 0; lo < (1 << half); lo++) {
                    const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                    inv_bfly(v[r0], v[r1], m[r0], m[r1], w, q);
                }
            }
        }
        const Tw fw = table_tw(cl, 2);
#pragma unroll
        for (int r = 0; r < NR / 2; r++) {
            u64 &x = v[r], &y = v[r + NR / 2];
            cap_to(x, m[r], 8, q);
            cap_to(y, m[r + NR / 2], 8, q);
            const u64 s = x + y, d = x + (q << 3) - y;
            x = canonical(mul4(s, f, q), 4, q);
            y = canonical(mul4(d, fw, q), 4, q);
        }
    }
}
// forward levels on `a` of values below 8 q: below 16 q
template <int RB>
__device__ __forceinline__ void fwd_columns(u64 (&v)[Col<RB>::NR], const ColTables<RB>& t, u64 q) {
    constexpr int NR = Col<RB>::NR, LV = Col<RB>::LEVELS;
    int m[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) m[r] = 8;
#pragma unroll
    for (int j = 0; j < LV; j++) {
        const int half = LV - 1 - j;
#pragma unroll
        for (int g = 0; g < (1 << j); g++) {
            const Tw w = t.at((1 << j) + g);
#pragma unroll
            for (int lo = 0; lo < (1 << half); lo++) {
                const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                fwd_bfly(v[r0], v[r1], m[r0], m[r1], w, q);
            }
        }
    }
    if constexpr (Col<RB>::SHARED) {
#pragma unroll
        for (int k = 0; k < NR / 2; k++) {
            swap_halves(v[2 * k], v[2 * k + 1]);
            m[2 * k] = m[2 * k + 1] = m[2 * k] > m[2 * k + 1] ? m[2 * k] : m[2 * k + 1];
            fwd_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], t.last(k), q);
        }
    }
}

// tasks: (polynomial, entry, tile of columns), one wave each
template <int K3, bool INV>
__device__ __forceinline__ void plain_columns(const IntArgs& a, const IntTasks& tk, int n_tasks) {
    constexpr int NR = Col<K3>::NR, TILES = Col<K3>::TILES;
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63, tile = task & (TILES - 1);
    const uint32_t unit = (uint32_t)task / TILES, e = uniform(unit / a.n_entries);
    const u64 b = unit - e * a.n_entries;
    const int prime = uniform(tk.prime[e]), pos = uniform(tk.pos[e]);
    const ModI q = mod_int(a.primes, prime);
    const ColTables<K3> t(INV ? a.itw : a.tw, INV ? a.itw_sh : a.tw_sh, prime, lane);
    const uint32_t first = column_lane<K3, true>(tile, lane), other = column_lane<K3, false>(tile, lane);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)pos * n, (uint32_t)n * 8u);
    u64 v[NR];
    if (INV) {
#pragma unroll
        for (int r = 0; r < NR; r++) v[r] = bload(dst, other, column_row<K3, false>(r));
        inv_columns<K3>(v, t, a.consts + (u64)prime * CONST_WORDS, q.q);
    } else {
        const rsrc_t src = a.coeffs ? make_rsrc(a.coeffs + b * n, (uint32_t)n * 8u)
                                    : make_rsrc(a.in + b * a.in_bs + (u64)(pos + a.in_pos_shift) * n, (uint32_t)n * 8u);
#pragma unroll
        for (int r = 0; r < NR; r++) v[r] = bload(src, first, column_row<K3, true>(r));
        if (a.coeffs) {                  // signed integers: reduce the magnitude
#pragma unroll
            for (int r = 0; r < NR; r++) {
                const bool neg = (i64)v[r] < 0;
                const u64 x = reduce4(neg ? 0 - v[r] : v[r], q);
                v[r] = neg ? (q.q << 2) - x : x;
            }
        }
        fwd_columns<K3>(v, t, q.q);
    }
#pragma unroll
    for (int r = 0; r < NR; r++) bstore(dst, INV ? first : other, column_row<K3, INV>(r), v[r]);
}

// One workgroup per (tile of columns, digit, share of the targets; entry).  ylds: [source of the chunk][NR][64 lanes], the
// conversion inputs as (y + floor(c / 2)) mod c in 30-bit halves: y's centred representative, shifted to be non-negative;
// `off` takes the shifts out of each target's sum again.
#define CONV_CHUNK 8     // terms below 2^60: sixteen of them fit the middle accumulator
template <int RB>
__device__ __forceinline__ void convert_columns(const IntArgs& a, u64* ylds) {
    constexpr int NR = Col<RB>::NR, TILES = Col<RB>::TILES, G = NR < 4 ? NR : 4;
    constexpr u64 n = (u64)1 << (10 + RB);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    const int tile = blockIdx.x & (TILES - 1), part = blockIdx.x / TILES, digit = part % a.n_digits, split = part / a.n_digits;
    const u64 b = blockIdx.y;
    const int src0 = digit * a.alpha, n_src = min(a.alpha, a.n_src - src0);
    const int own_n = a.own ? n_src : 0, n_tgt = a.ext_limbs - own_n;
    const int per_split = (n_tgt + a.n_splits - 1) / a.n_splits;
    const int t_first = split * per_split, t_end = min(t_first + per_split, n_tgt);
    const uint32_t first = column_lane<RB, true>(tile, lane), other = column_lane<RB, false>(tile, lane);
    const rsrc_t mid = make_rsrc(a.mid + (b * a.n_src + src0) * n, (uint32_t)(n_src * n * 8u));
    const int rounds = (t_end - t_first + waves - 1) / waves;
    const bool resident = n_src <= a.chunk;
    for (int round = 0; round < rounds; round++) {
        const int t = t_first + round * waves + wave;
        const bool mine = t < t_end;
        const int e = t < src0 || !own_n ? t : t + own_n;
        const int prime = mine ? prime_at(e, a.l, a.L) : 0;
        const ModI q = mod_int(a.primes, prime);
        const WideMod wide = wide_mod(a.consts, prime);
        const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)(digit * a.ext_limbs + (mine ? e : 0)) * n, (uint32_t)n * 8u);
        for (int c0 = 0; c0 < n_src; c0 += a.chunk) {
            const int c1 = min(c0 + a.chunk, n_src);
            if (!resident || round == 0) {
                if (c0 || round) __syncthreads();      // every wave is done with the chunk before
                for (int i = c0 + wave; i < c1; i += waves) {
                    const int sp = prime_at(a.src_pos0 + src0 + i, a.l, a.L);
                    const ModI qs = mod_int(a.primes, sp);
                    const u64 half = qs.q >> 1;
                    u64 w[NR];
#pragma unroll
                    for (int r = 0; r < NR; r++) w[r] = bload(mid, other, (uint32_t)(i * n * 8u) + column_row<RB, false>(r));
                    inv_columns<RB>(w, ColTables<RB>(a.itw, a.itw_sh, sp, lane), a.close + (u64)(src0 + i) * CLOSE_WORDS, qs.q);
                    u64* y = ylds + (i - c0) * NR * 64 + lane;
#pragma unroll
                    for (int r = 0; r < NR; r++) y[r * 64] = split30(sub_if(w[r] + half, qs.q));
                }
                __syncthreads();
            }
            if (!mine) continue;
            u64 v[NR];
            const u64 off = c0 ? 0 : as_constu(a.off)[(u64)digit * a.total + prime];
#pragma unroll
            for (int r0 = 0; r0 < NR; r0 += G) {
                Acc3 acc[G];
#pragma unroll
                for (int r = 0; r < G; r++) acc[r] = Acc3{off, 0, 0};
#pragma unroll 1
                for (int i = c0; i < c1; i++) {
                    const u64 hat = as_constu(a.hat)[(u64)(src0 + i) * a.total + prime];
                    const u64* y = ylds + ((i - c0) * NR + r0) * 64 + lane;
#pragma unroll
                    for (int r = 0; r < G; r++) acc3_mad(acc[r], y[r * 64], hat);
                }
#pragma unroll
                for (int r = 0; r < G; r++) v[r0 + r] = acc3_reduce(acc[r], wide, q.q);
                SCHED_FENCE();
            }
            if (c0) {                                  // partial sums of earlier chunks wait in the result's place
#pragma unroll
                for (int r = 0; r < NR; r++) v[r] = sub_if(v[r] + bload(dst, first, column_row<RB, true>(r)), q.q << 3);
            }
            if (c1 < n_src) {
#pragma unroll
                for (int r = 0; r < NR; r++) bstore(dst, first, column_row<RB, true>(r), v[r]);
                continue;
            }
            fwd_columns<RB>(v, ColTables<RB>(a.tw, a.tw_sh, prime, lane), q.q);
#pragma unroll
            for (int r = 0; r < NR; r++) bstore(dst, other, column_row<RB, false>(r), v[r]);
        }
    }
}

// ---------------------------------------------------------------------------
// the kernel family and its launches
// ---------------------------------------------------------------------------
template <int K3, int MODE, bool COLUMNS>
__global__ __launch_bounds__(COLUMNS && MODE == INT_CONVERT ? 512 : ROWS_NT,
                             COLUMNS && MODE == INT_CONVERT ? (K3 < 6 ? 4 : 2) : COLUMNS ? (K3 < 6 ? 4 : 2) : 6)
void ntt_int_kernel(IntArgs a, IntTasks tk, int n_tasks) {
    extern __shared__ u64 lds[];
    if constexpr (COLUMNS) {
        if constexpr (MODE == INT_CONVERT) convert_columns<K3>(a, lds);
        else plain_columns<K3, MODE == INT_INVERSE>(a, tk, n_tasks);
    } else {
        if constexpr (MODE == INT_INVERSE) rows_inverse<K3>(a, tk, n_tasks, lds);
        else if constexpr (MODE == INT_FORWARD) rows_forward<K3>(a, tk, n_tasks, lds);
        else if constexpr (MODE == INT_INNER) rows_inner<K3>(a, lds);
        else rows_divide<K3>(a, n_tasks, lds);
    }
}

template <int K3, int MODE>
__global__ __launch_bounds__(MODE == INT_INNER ? INNER_CHUNK * WIDE_NT : WIDE_NT, 4) void ntt_int_wide_kernel(IntArgs a, IntTasks tk, int n_tasks) {
    extern __shared__ u64 lds[];
    const int task = wide_task(n_tasks);
    if (task < 0) return;
    if constexpr (MODE == INT_INVERSE) wide_rows_inverse<K3>(a, tk, task, lds);
    else if constexpr (MODE == INT_INNER) wide_rows_inner<K3>(a, task, lds);
    else wide_rows_divide<K3>(a, task, lds);
}
template <int K3, int MODE>
static hipError_t launch_wide_k3(const IntArgs& a, const IntTasks& tk, u64 tasks, hipStream_t st) {
    static char name[40] = "";
    if (!name[0]) snprintf(name, sizeof name, "ntt_int_wide_kernel<%d, %d>", K3, MODE);
    IntArgs s = a;
    s.split = MODE == INT_INNER && 2 * tasks <= WIDE_SPLIT;
    const unsigned digits = (unsigned)a.n_digits, rows = MODE != INT_INNER ? 1 : s.split ? std::min(digits + 1, (unsigned)INNER_CHUNK) : std::max(digits, 2u);
    tasks <<= s.split;
    ProfScope prof__(name, st);
    hipLaunchKernelGGL((ntt_int_wide_kernel<K3, MODE>), dim3((unsigned)((tasks + 7) / 8 * 8)), dim3(rows * WIDE_NT), rows * WIDE_LDS * 8, st,
                       s, tk, (int)tasks);
    return hipGetLastError();
}
template <int MODE>
static hipError_t launch_wide(const IntArgs& a, const IntTasks& tk, u64 tasks, hipStream_t st) {
    switch (a.log_n) {
        case 10: return launch_wide_k3<0, MODE>(a, tk, tasks, st);
        case 11: return launch_wide_k3<1, MODE>(a, tk, tasks, st);
        case 12: return launch_wide_k3<2, MODE>(a, tk, tasks, st);
        case 13: return launch_wide_k3<3, MODE>(a, tk, tasks, st);
        case 14: return launch_wide_k3<4, MODE>(a, tk, tasks, st);
        case 15: return launch_wide_k3<5, MODE>(a, tk, tasks, st);
        case 16: return launch_wide_k3<6, MODE>(a, tk, tasks, st);
        default: return hipErrorInvalidValue;
    }
}

template <int K3, int MODE, bool COLUMNS>
static hipError_t launch_k3(dim3 grid, unsigned threads, size_t lds, const IntArgs& a, const IntTasks& tk, u64 tasks, hipStream_t st) {
    static char name[40] = "";      // what rocprofv3 prints for this instantiation
    static bool attr_set = false;
    if (!attr_set) {
        snprintf(name, sizeof name, "ntt_int_kernel<%d, %d, %s>", K3, MODE, COLUMNS ? "true" : "false");
        hipError_t e = hipFuncSetAttribute((const void*)ntt_int_kernel<K3, MODE, COLUMNS>, hipFuncAttributeMaxDynamicSharedMemorySize, 131072);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    ProfScope prof__(name, st);
    hipLaunchKernelGGL((ntt_int_kernel<K3, MODE, COLUMNS>), grid, dim3(threads), lds, st, a, tk, (int)tasks);
    return hipGetLastError();
}
template <int MODE, bool COLUMNS>
static hipError_t launch_any(int log_n, dim3 grid, unsigned threads, size_t lds, const IntArgs& a, const IntTasks& tk, u64 tasks, hipStream_t st) {
    switch (log_n) {
        case 10: return launch_k3<0, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 11: return launch_k3<1, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 12: return launch_k3<2, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 13: return launch_k3<3, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 14: return launch_k3<4, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 15: return launch_k3<5, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        case 16: return launch_k3<6, MODE, COLUMNS>(grid, threads, lds, a, tk, tasks, st);
        default: return hipErrorInvalidValue;
    }
}
// Rows by four waves or by one.  Inverse rows: 8 rows 8.5 -> 4.7 us, 512 rows 10 -> 6.3, 4096 rows 29 -> 25; with the columns behind
// them 32768 rows 228 -> 226 us at N = 2^15, but 49152 rows there 386 -> 392 and 65536 rows 516 -> 520, 131072 rows at 2^12 988 -> 1010
// (at 2^10, where the rows are all there is, either within 2 % from 16384 rows on).  Rows of a division: 24 rows 10.3 -> 5.2 us, 1024 rows 15 -> 9.7, 8192 rows 63 -> 62, but 32768 rows 223 -> 247:
// the wave of its own waits for fewer exchanges.  Inner products: while all workgroups are resident at once, 512 of eight
// waves (up to two digits) or 256 of twelve or sixteen: one wave a digit -> four, 16 tasks of three digits 17.6 -> 12.8 us, 256 of
// them 18.5 -> 14.4, 352 23 -> 26; of two digits 512 tasks 22 -> 17.6, 768 24.7 -> 24.3, 1024 29 -> 30.
// Of these a workgroup for each polynomial while both fit the chip's 256 compute units (WIDE_SPLIT): one rotation at N = 2^12,
// 3 limbs, 28.4 -> 28.0 us; with 6 .. 48 tasks of two digits at N = 2^10 25.8 .. 26.4 -> 24.7 .. 25.4, with 128 of three digits at N = 2^12
// 31.1 -> 29.9; 144 and 192 tasks as without.
#define WIDE_INVERSE_ROWS 32768
#define WIDE_DIVIDE_ROWS 8192
static u64 wide_inner_tasks(int n_digits) { return n_digits > INNER_CHUNK ? 0 : n_digits <= 2 ? 512 : 256; }

template <int MODE, bool COLUMNS>
static hipError_t launch_waves(const IntArgs& a, const IntTasks& tk, u64 tasks, hipStream_t st) {
    if (tasks > 0x7fffff00u) return hipErrorInvalidValue;
    if constexpr (MODE == INT_INVERSE && !COLUMNS)
        if (tasks <= WIDE_INVERSE_ROWS) return launch_wide<MODE>(a, tk, tasks, st);
    const u64 blocks = ((tasks + ROWS_NT / 64 - 1) / (ROWS_NT / 64) + 7) / 8 * 8;
    const size_t lds = COLUMNS ? 0 : (size_t)(ROWS_NT / 64) * ROW_LDS * 8;
    return launch_any<MODE, COLUMNS>(a.log_n, dim3((unsigned)blocks), ROWS_NT, lds, a, tk, tasks, st);
}
static hipError_t launch_inner(const IntArgs& a, hipStream_t st) {
    const u64 tasks = ((u64)a.ext_limbs * a.n_entries) << (a.log_n - 10);
    if (tasks <= wide_inner_tasks(a.n_digits)) return launch_wide<INT_INNER>(a, IntTasks{}, tasks, st);
    const int slots = a.n_digits < 2 ? 2 : a.n_digits < INNER_CHUNK ? a.n_digits : INNER_CHUNK;
    const uint32_t parts = inner_parts(a.log_n - 10);             // a workgroup per task, eight times what the first XCD takes
    const u64 blocks = (u64)((a.ext_limbs + parts - 1) / parts * inner_rows(a.log_n - 10)) * a.n_entries * 8;
    if (blocks > 0x7fffff00u) return hipErrorInvalidValue;
    return launch_any<INT_INNER, false>(a.log_n, dim3((unsigned)blocks), slots == 2 ? 128 : ROWS_NT, (size_t)slots * ROW_LDS * 8, a,
                                        IntTasks{}, tasks, st);
}

static bool base_ok(const IntArgs& a) {
    return a.log_n >= 10 && a.log_n <= 16 && a.primes && a.tw && a.tw_sh && a.itw && a.itw_sh && a.consts && a.n_entries >= 1;
}
static bool tasks_ok(const IntTasks& tk) {
    if (tk.n < 1 || tk.n > HISA_MAX_PERIOD) return false;
    for (int i = 0; i < tk.n; i++)
        if (tk.prime[i] < 0 || tk.pos[i] < 0) return false;
    return true;
}

hipError_t launch_ntt_int(const IntArgs& a, const IntTasks& tk, hipStream_t st) {
    DRY_RUN_RETURN();
    if (!base_ok(a) || !tasks_ok(tk) || !a.out || (!a.in && !a.coeffs)) return hipErrorInvalidValue;
    const u64 polys = (u64)tk.n * a.n_entries;
    if (a.log_n > 10 || a.coeffs) {
        hipError_t e = launch_waves<INT_FORWARD, true>(a, tk, polys * (a.log_n < 15 ? 16 : 32), st);
        if (e != hipSuccess) return e;
    }
    return launch_waves<INT_FORWARD, false>(a, tk, polys << (a.log_n - 10), st);
}

hipError_t launch_intt_int(const IntArgs& a_in, const IntTasks& tk, hipStream_t st) {
    DRY_RUN_RETURN();
    IntArgs a = a_in;
    a.whole = 1;
    if (!base_ok(a) || !tasks_ok(tk) || !a.out || !a.in) return hipErrorInvalidValue;
    const u64 polys = (u64)tk.n * a.n_entries;
    hipError_t e = launch_waves<INT_INVERSE, false>(a, tk, polys << (a.log_n - 10), st);
    return e != hipSuccess || a.log_n == 10 ? e : launch_waves<INT_INVERSE, true>(a, tk, polys * (a.log_n < 15 ? 16 : 32), st);
}

hipError_t launch_inverse_rows_int(const IntArgs& a_in, hipStream_t st) {
    DRY_RUN_RETURN();
    IntArgs a = a_in;
    IntTasks tk;
    if (!base_ok(a) || !a.in || !a.mid || a.n_src < 1 || a.n_src > HISA_MAX_PERIOD || a.src_pos0 < 0) return hipErrorInvalidValue;
    for (int k = 0; k < a.n_src; k++) {
        const int pos = a.src_pos0 + k, prime = pos < a.l ? pos : pos + (a.L - a.l);
        if (prime >= a.total) return hipErrorInvalidValue;
        tk.pos[k] = (int16_t)k;
        tk.prime[k] = (int16_t)prime;
    }
    tk.n = a.n_src;
    a.in_pos_shift = a.src_pos0;
    a.out = a.mid; a.out_bs = (u64)a.n_src << a.log_n;
    a.whole = 0;
    return launch_waves<INT_INVERSE, false>(a, tk, ((u64)a.n_src * a.n_entries) << (a.log_n - 10), st);
}

static bool convert_ok(const IntArgs& a) {
    return base_ok(a) && a.mid && a.out && a.close && a.hat && a.off && a.n_src >= 1 && a.alpha >= 1 && a.src_pos0 >= 0 && a.l >= 1 && a.L >= a.l &&
           a.n_digits >= 1 && (a.n_digits - 1) * a.alpha < a.n_src && a.n_digits * a.alpha >= a.n_src && a.ext_limbs >= 1 &&
           a.ext_limbs - a.l + a.L <= a.total && a.n_entries <= 65535 && (!a.own || (a.src_pos0 == 0 && a.n_src <= a.ext_limbs));
}

// Waves of a workgroup of the columns where there are twice as many workgroups as are resident with eight waves each: those with the
// highest throughput of the workgroups that there are (few waves leave room for more than those: 8 rotations at N = 2^16, 4 limbs, two
// digits, in 512 workgroups of two waves 181 us, of four 157), when `slots` waves share a compute unit and a round over the targets takes
// 1.6 times one over the sources.  A wave without a target in the last round, or without a source, only holds its registers, and those
// admit seven waves a SIMD up to N = 2^13, four at 2^14 and 2^15, two at 2^16 (tests/test_kernel_registers_host.py).  rotLeft, us, as few
// waves as the rounds need (five, of 9 targets and 3 sources) -> these (three): 16 at N = 2^15, 8 limbs, three digits 331 -> 320, 64 at N = 2^14
// 564 -> 538, 16 at N = 2^16, 4 limbs, two digits 321 -> 299, 64 at N = 2^11, 7 limbs 79 -> 76; even where the waves stay.  With fewer
// workgroups the rounds are what counts: 12 at N = 2^15, 5 limbs, in 768 workgroups 163 -> 174.
static int columns_waves(const IntArgs& a, size_t lds, int slots, u64 workgroups) {
    int best = 8;
    double best_rate = 0;
    for (int w = 2; w <= 8; w++) {
        double time = 0;
        for (int d = 0; d < a.n_digits; d++) {
            const int src = std::min(a.alpha, a.n_src - d * a.alpha), tgt = a.ext_limbs - (a.own ? src : 0);
            time += (src + w - 1) / w + 1.6 * ((tgt + w - 1) / w);
        }
        const double rate = std::min({(double)(slots / w), (double)(163840 / lds), workgroups / 256.0}) / time;
        if (rate > best_rate) { best_rate = rate; best = w; }
    }
    return best;
}

hipError_t launch_columns_int(const IntArgs& a_in, hipStream_t st) {
    DRY_RUN_RETURN();
    IntArgs a = a_in;
    if (!convert_ok(a)) return hipErrorInvalidValue;
    const int most_src = a.alpha < a.n_src ? a.alpha : a.n_src, last_src = a.n_src - (a.n_digits - 1) * a.alpha;
    const int most_tgt = a.ext_limbs - (a.own ? last_src : 0);
    if (most_tgt < 1) return hipSuccess;
    const unsigned tiles = a.log_n < 15 ? 16 : 32;               // Col::TILES, and a source's words in LDS
    const size_t per_src = (size_t)512 << (a.log_n < 15 ? a.log_n - 10 : a.log_n - 11);
    const int fit = (int)(131072 / per_src), limit = fit < CONV_CHUNK ? fit : CONV_CHUNK;
    a.chunk = most_src < limit ? most_src : limit;
    // a target per wave, and as few waves as the rounds over the targets need
    const int rounds = (most_tgt + 7) / 8;
    int waves = (most_tgt + rounds - 1) / rounds;
    const int slots = a.log_n < 14 ? 28 : a.log_n < 16 ? 16 : 8;
    const u64 workgroups = (u64)a.n_entries * a.n_digits * tiles;
    if (most_src <= a.chunk && workgroups >= 64u * slots) waves = columns_waves(a, a.chunk * per_src, slots, workgroups);
    // few entries: several workgroups share a tile's targets (each forms the conversion inputs for itself)
    a.n_splits = 1;
    while (a.n_splits < rounds && (u64)a.n_entries * a.n_digits * tiles * (a.n_splits + 1) <= 512) a.n_splits++;
    return launch_any<INT_CONVERT, true>(a.log_n, dim3(tiles * (unsigned)(a.n_digits * a.n_splits), a.n_entries), (unsigned)waves * 64,
                                         a.chunk * per_src, a, IntTasks{}, 0, st);
}

hipError_t launch_divide_rows_int(const IntArgs& a, hipStream_t st) {
    DRY_RUN_RETURN();
    if (!convert_ok(a) || a.n_digits != 1 || a.own || !a.acc || !a.factor || !a.factor_sh || a.ext_limbs > a.l || (a.add && a.add_div < 1))
        return hipErrorInvalidValue;
    const u64 rows = ((u64)a.ext_limbs * a.n_entries) << (a.log_n - 10);
    return rows <= WIDE_DIVIDE_ROWS ? launch_wide<INT_CONVERT>(a, IntTasks{}, rows, st) : launch_waves<INT_CONVERT, false>(a, IntTasks{}, rows, st);
}

hipError_t launch_inner_rows_int(const IntArgs& a, hipStream_t st) {
    DRY_RUN_RETURN();
    if (!base_ok(a) || !a.in || !a.ext || !a.key || !a.sums || !a.down || a.alpha < 1 || a.n_digits < 1 || a.n_digits * a.alpha < a.l ||
        (a.n_digits - 1) * a.alpha >= a.l || a.ext_limbs <= a.l || a.ext_limbs - a.l + a.L > a.total)
        return hipErrorInvalidValue;
    return launch_inner(a, st);
}
