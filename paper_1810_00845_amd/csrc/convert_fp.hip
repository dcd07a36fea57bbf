// Inverse transform -> fast base conversion -> forward transform, in exact fp64, for N = 2^12 .. 2^15 and primes below
// 2^50: the ModUp and the ModDown of key switching and the division of a rescale, as three launches whose units of
// work are single waves (rows) or small workgroups (columns).
//
// A coefficient index is (a : log2 N - 10)(b : 5)(c : 5).  The log2 N - 10 levels on `a` pair coefficients a multiple
// of 1024 apart ("columns"), the ten levels on b and c stay inside a row of 1024 neighbours.
//   rows_inv     one wave per row: the inverse levels on c, then b
//   columns      one workgroup per tile of columns of one digit of one entry: the inverse levels on `a` of all its source
//                limbs (-> centred conversion inputs, kept in LDS), then per target limb the conversion sum and the
//                forward levels on `a`
//   rows_fwd     one wave per row: the forward levels on b, then c, and the store stage of the operation
// Why this split: a workgroup that transforms a whole polynomial (ntt_fp.hip) occupies one compute unit for 20-36 us
// whatever else is idle, so a call with fewer limb-polynomials than compute units is bound by that latency.  Here a
// polynomial at N = 2^15 is 32 waves of rows and 32 tiles of columns, nothing waits for a whole polynomial except
// the launch boundary, and the conversion inputs never travel through memory.  rotLeft against whole-polynomial workgroups
// (which also sent the extended digits through memory once more): 64 ciphertexts at N = 2^15, 16 limbs, 1.84 -> 1.28 ms;
// 3 at 17 limbs 223 -> 107 us; one at N = 2^13, 8 limbs, 64 -> 26 us.  Large batches are bound by fp64 issue in the columns
// and by memory in the rows, single ciphertexts by five launches of 4-8 us, each a chain of dependent levels.
//
// A wave holds 1024 coefficients, 16 per lane.  Five levels on a five-bit field take four in registers and the one on
// the field's lowest bit after exchanging that bit (lane bit 5) with a register bit by v_permlane32_swap; those on b take
// three in registers and two behind exchanges, since a lane's register pairs are neighbours in memory.  A row needs
// two passes through LDS in all (one 64-bit exchange each way) and loads and stores are whole kilobytes.
//
// Ranges: values are exact integers |v| <= m p with m p < 2^53; every butterfly knows the bound m of its operands at
// compile time (Bound below: plain floats that fold away after unrolling) and normalises only where the result could
// leave 8 p.
#include <cstdio>
#include <type_traits>

#include "fp_device.hpp"
#include "modarith.hpp"
#include "sampling.hpp"

#define HEAD 64          // per-prime table: [HEAD] column twiddles, then SPLIT_ROW per row (layout: split_tables)

struct Modulus { double p, pinv; };
__device__ __forceinline__ Modulus modulus(const FpPrime* f, int prime) {
    return Modulus{as_const(&f[prime].p)[0], as_const(&f[prime].p)[1]};
}

#define BOUND_LIMIT 7.99f
__device__ __forceinline__ float product_bound(float my, float mw) { return 0.501f + 0.375f * my * mw; }   // fp_mulmod

// forward butterfly: (x, y) -> (x + w y, x - w y)
__device__ __forceinline__ void fwd_bfly(double& x, double& y, float& bx, float& by, double w, float mw, Modulus q) {
    const float bt = product_bound(by, mw);
    if (bx + bt > BOUND_LIMIT) { x = fp_norm(x, q.p, q.pinv); bx = 0.501f; }
    const double t = fp_mulmod(y, w, q.p, q.pinv);
    y = x - t;
    x = x + t;
    bx = by = bx + bt;
}

// inverse butterfly: (x, y) -> (x + y, (x - y) w)
__device__ __forceinline__ void inv_bfly(double& x, double& y, float& bx, float& by, double w, float mw, Modulus q) {
    if (bx + by > BOUND_LIMIT) {
        x = fp_norm(x, q.p, q.pinv);
        y = fp_norm(y, q.p, q.pinv);
        bx = by = 0.501f;
    }
    const double d = x - y;
    x = x + y;
    bx = bx + by;
    y = fp_mulmod(d, w, q.p, q.pinv);
    by = product_bound(bx, mw);
}

// exchange lane bit 5 with the register bit that tells x from y: afterwards x holds what the lanes of the lower half had
// in (x, y), y what those of the upper half had
__device__ __forceinline__ void swap_halves(double& x, double& y) {
    const auto lo = __builtin_amdgcn_permlane32_swap(lo32(x), lo32(y), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(hi32(x), hi32(y), false, false);
    x = mk64(lo[0], hi[0]);
    y = mk64(lo[1], hi[1]);
}

// the same for lane bit 4
__device__ __forceinline__ void swap_quarters(double& x, double& y) {
    const auto lo = __builtin_amdgcn_permlane16_swap(lo32(x), lo32(y), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(hi32(x), hi32(y), false, false);
    x = mk64(lo[0], hi[0]);
    y = mk64(lo[1], hi[1]);
}

// Five forward levels on a five-bit field.  In: register r of a lane in half h holds element 2 r + h; out: element
// 4 (r >> 1) + 2 h + (r & 1).  tw(j, g): twiddle of level j < 4, group g; last[k]: of level 4, group 2 k + h.
template <class TW>
__device__ __forceinline__ void fwd_levels5(double (&v)[16], float (&m)[16], TW tw, float mw, const double (&last)[8], Modulus q) {
#pragma unroll
    for (int j = 0; j < 4; j++) {
        const int half = 3 - j;
#pragma unroll
        for (int g = 0; g < (1 << j); g++) {
            const double w = tw(j, g);
#pragma unroll
            for (int lo = 0; lo < (1 << half); lo++) {
                const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                fwd_bfly(v[r0], v[r1], m[r0], m[r1], w, mw, q);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        swap_halves(v[2 * k], v[2 * k + 1]);
        m[2 * k] = m[2 * k + 1] = fmaxf(m[2 * k], m[2 * k + 1]);
        fwd_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], last[k], 0.5f, q);
    }
}

// The inverse levels, undone in reverse order.  In: element 4 (r >> 1) + 2 h + (r & 1); out: 2 r + h.
template <class TW>
__device__ __forceinline__ void inv_levels5(double (&v)[16], float (&m)[16], TW tw, float mw, const double (&last)[8], Modulus q,
                                            int lowest_level = 0) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
        inv_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], last[k], 0.5f, q);
        swap_halves(v[2 * k], v[2 * k + 1]);
        m[2 * k] = m[2 * k + 1] = fmaxf(m[2 * k], m[2 * k + 1]);
    }
#pragma unroll
    for (int j = 3; j >= 0; j--) {
        if (j < lowest_level) continue;
        const int half = 3 - j;
#pragma unroll
        for (int g = 0; g < (1 << j); g++) {
            const double w = tw(j, g);
#pragma unroll
            for (int lo = 0; lo < (1 << half); lo++) {
                const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                inv_bfly(v[r0], v[r1], m[r0], m[r1], w, mw, q);
            }
        }
    }
}

// the largest bound of all registers becomes everyone's (values change lanes and registers in an exchange); what could
// be larger than `cap` is normalised first
__device__ __forceinline__ void cap_bounds(double (&v)[16], float (&m)[16], float cap, Modulus q) {
    float top = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r++) {
        if (m[r] > cap) { v[r] = fp_norm(v[r], q.p, q.pinv); m[r] = 0.501f; }
        top = fmaxf(top, m[r]);
    }
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = top;
}

// The five levels on b of a row whose neighbouring coefficients share a lane: register 2 k + p of lane i holds element
// b = 4 k + (i >> 4) of column c = 2 (i & 15) + p, so that the row is loaded and stored in 16-byte accesses (rows_inner tells
// why).  Three levels in registers; the one on bit 1 of b behind an exchange of it (lane bit 5) with the register bit p, the one
// on bit 0 behind an exchange (lane bit 4) with that register bit again.  Out: element 4 k + 2 (lane bit 4) + p of column
// 2 (i & 15) + (lane bit 5).  last[k]: twiddle of level 4, group 2 k + (lane bit 4).
__device__ __forceinline__ void unify(float& a, float& b) { a = b = fmaxf(a, b); }
template <class TW>
__device__ __forceinline__ void fwd_levels_b(double (&v)[16], float (&m)[16], TW tw, const double (&last)[8], Modulus q) {
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const int half = 2 - j;
#pragma unroll
        for (int g = 0; g < (1 << j); g++) {
            const double w = tw(j, g);
#pragma unroll
            for (int lo = 0; lo < (2 << half); lo++) {
                const int r0 = (g << (half + 2)) | lo, r1 = r0 + (2 << half);
                fwd_bfly(v[r0], v[r1], m[r0], m[r1], w, 0.5f, q);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        swap_halves(v[2 * k], v[2 * k + 1]);
        unify(m[2 * k], m[2 * k + 1]);
        fwd_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], tw(3, k), 0.5f, q);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        swap_quarters(v[2 * k], v[2 * k + 1]);
        unify(m[2 * k], m[2 * k + 1]);
        fwd_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], last[k], 0.5f, q);
    }
}
template <class TW>
__device__ __forceinline__ void inv_levels_b(double (&v)[16], float (&m)[16], TW tw, const double (&last)[8], Modulus q) {
#pragma unroll
    for (int k = 0; k < 8; k++) {
        inv_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], last[k], 0.5f, q);
        swap_quarters(v[2 * k], v[2 * k + 1]);
        unify(m[2 * k], m[2 * k + 1]);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        inv_bfly(v[2 * k], v[2 * k + 1], m[2 * k], m[2 * k + 1], tw(3, k), 0.5f, q);
        swap_halves(v[2 * k], v[2 * k + 1]);
        unify(m[2 * k], m[2 * k + 1]);
    }
#pragma unroll
    for (int j = 2; j >= 0; j--) {
        const int half = 2 - j;
#pragma unroll
        for (int g = 0; g < (1 << j); g++) {
            const double w = tw(j, g);
#pragma unroll
            for (int lo = 0; lo < (2 << half); lo++) {
                const int r0 = (g << (half + 2)) | lo, r1 = r0 + (2 << half);
                inv_bfly(v[r0], v[r1], m[r0], m[r1], w, 0.5f, q);
            }
        }
    }
}
// Words of a row in LDS.  In order: coefficient i at i + i / 32; of register 2 k + p: row_at + 132 k + p.  Between the levels on
// b and on c: element b of column c at 33 rho(b) + c / 2 + 16 (c & 1), rho putting bit 1 of b on top, which spreads what the
// lanes of either side touch over all banks; of register r before the levels on c: mid_c + r, of register r behind those on b: mid_b + 33 r.
__device__ __forceinline__ int row_at(int lane) { return 33 * (lane >> 4) + 2 * (lane & 15); }
__device__ __forceinline__ int mid_b(int lane) { return 528 * ((lane >> 4) & 1) + (lane & 15) + 16 * (lane >> 5); }
__device__ __forceinline__ int mid_c(int lane) {
    const int b = lane & 31;
    return 33 * (((b & 2) << 3) | ((b >> 2) << 1) | (b & 1)) + 16 * (lane >> 5);
}
#define ROW_REG(r) (132 * ((r) >> 1) + ((r) & 1))

// What a wave keeps of the twiddles of its row (layout: split_table_words)
struct RowTwiddles {
    double last_c[8], last_b[8], base[4];
    const double *head, *tab;
};
__device__ __forceinline__ void row_tables(RowTwiddles& w, const double* table, u64 stride, int prime, uint32_t row) {
    w.head = table + (u64)prime * stride;
    w.tab = w.head + HEAD + (u64)row * SPLIT_ROW;
}
__device__ __forceinline__ void load_twiddles_b(RowTwiddles& w, int lane) {
    const rsrc_t r = make_rsrc(w.tab, SPLIT_ROW * 8);
#pragma unroll
    for (int k = 0; k < 4; k++) bload2(r, (uint32_t)((lane >> 4) & 1) * 64u, 128u + (uint32_t)k * 16u, w.last_b[2 * k], w.last_b[2 * k + 1]);
}
__device__ __forceinline__ void load_twiddles_c(RowTwiddles& w, int lane) {
    const rsrc_t r = make_rsrc(w.tab, SPLIT_ROW * 8);
#pragma unroll
    for (int k = 0; k < 4; k++) bload2(r, (uint32_t)lane * 16u, 160u * 8u + (uint32_t)k * 1024u, w.last_c[2 * k], w.last_c[2 * k + 1]);
#pragma unroll
    for (int j = 0; j < 4; j++) w.base[j] = bloadf(r, (uint32_t)(lane & 31) * 8u, 32u * 8u + (uint32_t)j * 256u);
}
__device__ __forceinline__ void load_row_twiddles(RowTwiddles& w, const double* table, u64 stride, int prime, uint32_t row, int lane) {
    row_tables(w, table, stride, prime, row);
    load_twiddles_c(w, lane);
    load_twiddles_b(w, lane);
}

// The ten levels of a row; register 2 k + p of lane i is coefficient 128 k + 2 i + p before and after.  m: bounds, in and out.
// LATE: the twiddles of c are fetched behind the levels on b (a caller short of registers).  LEAVE: the result stays in
// the wave's LDS part, in order.
template <bool LATE = false, bool LEAVE = false>
__device__ __forceinline__ void row_forward(double (&v)[16], float (&m)[16], RowTwiddles& w, double* lds, int lane, Modulus q, float cap) {
    const int h = lane >> 5, s = lane & 31;
    fwd_levels_b(v, m, [&](int j, int g) { return as_const(w.tab)[(1 << j) + g]; }, w.last_b, q);
    cap_bounds(v, m, BOUND_LIMIT, q);
    if (LATE) {
        SCHED_FENCE();
        load_twiddles_c(w, lane);
    }
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[mid_b(lane) + 33 * r] = v[r];
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[mid_c(lane) + r];
    fwd_levels5(v, m, [&](int j, int g) { return g == 0 ? w.base[j] : fp_mulmod(w.base[j], as_const(w.head)[32 + g], q.p, q.pinv); },
                0.6f, w.last_c, q);
    cap_bounds(v, m, cap, q);
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[s * 33 + 2 * h + (r >> 1) * 4 + (r & 1)] = v[r];
    if (LEAVE) return;
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[row_at(lane) + ROW_REG(r)];
}

__device__ __forceinline__ void row_inverse(double (&v)[16], float (&m)[16], RowTwiddles& w, double* lds, int lane, Modulus q) {
    const int h = lane >> 5, s = lane & 31;
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[row_at(lane) + ROW_REG(r)] = v[r];
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[s * 33 + 2 * h + (r >> 1) * 4 + (r & 1)];     // lane b = s, elements of c
    inv_levels5(v, m, [&](int j, int g) { return g == 0 ? w.base[j] : fp_mulmod(w.base[j], as_const(w.head)[32 + g], q.p, q.pinv); },
                0.6f, w.last_c, q);
    cap_bounds(v, m, 2.01f, q);
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) lds[mid_c(lane) + r] = v[r];
    xchg_sync<true>();
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = lds[mid_b(lane) + 33 * r];
    inv_levels_b(v, m, [&](int j, int g) { return as_const(w.tab)[(1 << j) + g]; }, w.last_b, q);
    cap_bounds(v, m, 1.01f, q);
}

__device__ __forceinline__ void load_row(double (&v)[16], rsrc_t row, int lane) {
#pragma unroll
    for (int k = 0; k < 8; k++) bload2(row, (uint32_t)lane * 16u, (uint32_t)k * 1024u, v[2 * k], v[2 * k + 1]);
}
template <bool ONCE>
__device__ __forceinline__ void load_key_row(double (&v)[16], rsrc_t row, int lane) {
    if (!ONCE) return load_row(v, row, lane);
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const u32x4_t d = __builtin_amdgcn_raw_buffer_load_b128(row, lane * 16, k * 1024, NONTEMPORAL);
        v[2 * k] = mk64(d.x, d.y);
        v[2 * k + 1] = mk64(d.z, d.w);
    }
}
__device__ __forceinline__ void store_row(rsrc_t row, int lane, const double (&v)[16]) {
#pragma unroll
    for (int k = 0; k < 8; k++) bstore2(row, (uint32_t)lane * 16u, (uint32_t)k * 1024u, v[2 * k], v[2 * k + 1]);
}
__device__ __forceinline__ void from_residues(double (&v)[16]) {
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = fp_from_u64((u64)__double_as_longlong(v[r]));
}
__device__ __forceinline__ void store_residues(rsrc_t row, int lane, double (&v)[16], Modulus q) {
#pragma unroll
    for (int r = 0; r < 16; r++) v[r] = __longlong_as_double((long long)fp_canonical(v[r], q.p, q.pinv));
    store_row(row, lane, v);
}

// the row's 1024 words of a limb, read through sigma_g when galois != 0: neighbours come from a pair of neighbours, in either
// order (their exponents are N apart, and stay so under an odd factor)
template <int K3>
__device__ __forceinline__ void load_row_through(double (&v)[16], const u64* limb, u64 galois, uint32_t row, int lane) {
    if (galois) {
        const rsrc_t src = make_rsrc(limb, (uint32_t)8192 << K3);
        const Gather t = make_gather(galois, row, 2 * lane, 10 + K3);
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t at = gather_offset(t, 2 * k);
            double x, y;
            bload2(src, at & ~8u, 0, x, y);
            const bool turned = (at & 8u) != 0;
            v[2 * k] = turned ? y : x;
            v[2 * k + 1] = turned ? x : y;
        }
    } else {
        load_row(v, make_rsrc(limb + row * 1024u, 8192u), lane);
    }
}

// ---------------------------------------------------------------------------
// rows, inverse
// ---------------------------------------------------------------------------
template <int K3>
__device__ __forceinline__ void rows_inverse(const ConvertArgs& a, int n_tasks, double* lds_all) {
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    double* lds = lds_all + (threadIdx.x >> 6) * ROW_LDS;
    const uint32_t unit = (uint32_t)task / a.n_entries, b = (uint32_t)task - unit * a.n_entries;
    const uint32_t row = unit & ((1u << K3) - 1), k = unit >> K3;
    const int prime = prime_at(a.src_pos0 + (int)k, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    double v[16];
    float m[16];
    const u64* src_p = a.in + (u64)b * a.in_bs + (u64)(a.src_pos0 + (int)k) * n;
    load_row_through<K3>(v, src_p, a.galois, row, lane);
    RowTwiddles w;
    load_row_twiddles(w, a.sinv, a.table_stride, prime, row, lane);
    from_residues(v);
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = 1.0f;
    row_inverse(v, m, w, lds, lane, q);
    store_row(make_rsrc(a.mid + ((u64)b * a.n_src + k) * n + row * 1024u, 8192u), lane, v);
}

// ---------------------------------------------------------------------------
// columns
// ---------------------------------------------------------------------------
// Bound by fp64 issue beside memory: 64 rotations at N = 2^15, 16 limbs, with the products and levels left out the launch over
// the digits takes 207 us (its bytes), with the stores left out 240 us, whole 265 us.  Its conversion sums are FpSums: products
// reduced one by one made it 305 us, those of the division by P 208 us against 183 now.  The sums are not held over the sources'
// levels, so that 80 registers do and three workgroups share a compute unit (277 us with two; without the limit the compiler takes
// 81, so seven sources and more, whose LDS admits two workgroups, lose nothing by it).  Only digits of more sources than the LDS holds
// keep them, in 92 registers (HELD below): 64 rotations at N = 2^15, 21 limbs, one digit, 2228 us against 2342 with the sums in memory
// between chunks, 16 at N = 2^14, 24 limbs, 318 against 348.
template <int RB>
struct Col {
    static constexpr int NR = RB == 5 ? 16 : (1 << RB);      // coefficients per lane
    static constexpr int WIDTH = RB == 5 ? 32 : 64;          // columns per tile
};

// Inverse levels on `a`, the last one with the limb's factor f folded in.  RB = 5: in / out elements as inv_levels5.
template <int RB>
__device__ __forceinline__ void inv_columns(double (&v)[Col<RB>::NR], const double* head, const double (&last)[8], double f, double fw,
                                            Modulus q) {
    constexpr int NR = Col<RB>::NR;
    float m[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) m[r] = 1.01f;
    if constexpr (RB == 5) {
        inv_levels5(v, m, [&](int j, int g) { return as_const(head)[(1 << j) + g]; }, 0.5f, last, q, 1);
    } else {
#pragma unroll
        for (int j = RB - 1; j >= 1; j--) {
            const int half = RB - 1 - j;
#pragma unroll
            for (int g = 0; g < (1 << j); g++)
#pragma unroll
                for (int lo = 0; lo < (1 << half); lo++) {
                    const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                    inv_bfly(v[r0], v[r1], m[r0], m[r1], as_const(head)[(1 << j) + g], 0.5f, q);
                }
        }
    }
#pragma unroll
    for (int r = 0; r < NR / 2; r++) {
        double &x = v[r], &y = v[r + NR / 2];
        if (m[r] + m[r + NR / 2] > BOUND_LIMIT) { x = fp_norm(x, q.p, q.pinv); y = fp_norm(y, q.p, q.pinv); }
        const double s = x + y, d = x - y;
        x = fp_norm(fp_mulmod(s, f, q.p, q.pinv), q.p, q.pinv);
        y = fp_norm(fp_mulmod(d, fw, q.p, q.pinv), q.p, q.pinv);
    }
}

template <int RB>
__device__ __forceinline__ void fwd_columns(double (&v)[Col<RB>::NR], const double* head, const double (&last)[8], Modulus q) {
    constexpr int NR = Col<RB>::NR;
    float m[NR];
#pragma unroll
    for (int r = 0; r < NR; r++) m[r] = 0.501f;
    if constexpr (RB == 5) {
        fwd_levels5(v, m, [&](int j, int g) { return as_const(head)[(1 << j) + g]; }, 0.5f, last, q);
    } else {
#pragma unroll
        for (int j = 0; j < RB; j++) {
            const int half = RB - 1 - j;
#pragma unroll
            for (int g = 0; g < (1 << j); g++)
#pragma unroll
                for (int lo = 0; lo < (1 << half); lo++) {
                    const int r0 = (g << (half + 1)) | lo, r1 = r0 + (1 << half);
                    fwd_bfly(v[r0], v[r1], m[r0], m[r1], as_const(head)[(1 << j) + g], 0.5f, q);
                }
        }
    }
}
#define COLUMNS_BOUND 4.85f   // of the stored values: five levels from normalised sums

// ylds: [source of the chunk][NR][64 lanes].  HELD: the sources come in several chunks, and a target's sums stay in registers from one
// to the next; else they are all in LDS.
template <int RB, bool HELD>
__device__ __forceinline__ void columns(const ConvertArgs& a, double* ylds) {
    constexpr int NR = Col<RB>::NR, WIDTH = Col<RB>::WIDTH, TILES = 1024 / WIDTH;
    const int lane = threadIdx.x & 63, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), waves = (int)(blockDim.x >> 6);
    const int tile = blockIdx.x & (TILES - 1), part = blockIdx.x / TILES, digit = part % a.n_digits, split = part / a.n_digits;
    constexpr u64 n = (u64)1 << (10 + RB);
    const u64 b = blockIdx.y;
    const int src0 = a.dg[digit].src0, n_src = a.dg[digit].a, own_lo = a.dg[digit].own_lo, own_n = a.dg[digit].own_n;
    const int n_tgt = a.ext_limbs - own_n;
    const int per_split = (n_tgt + a.n_splits - 1) / a.n_splits;
    const int t_first = split * per_split, t_end = min(t_first + per_split, n_tgt);
    const int col = tile * WIDTH + (RB == 5 ? (lane & 31) : lane);
    // lane part and register part of a row's address before the forward / after the inverse levels; RB = 5 keeps two rows
    // per register, one in each half of the wave
    const uint32_t in_lane = (uint32_t)((RB == 5 ? 2 * h * 1024 : 0) + col) * 8u;
    const rsrc_t mid = make_rsrc(a.mid + (b * a.n_src + src0) * n, (uint32_t)(n_src * n * 8u));
    const int rounds = (t_end - t_first + waves - 1) / waves;
    const int chunk = HELD ? a.chunk : n_src;
    const bool resident = n_src <= chunk;
    for (int round = 0; round < rounds; round++) {
        const int t = t_first + round * waves + wave;
        const bool mine = t < t_end;
        const int e = t < own_lo ? t : t + own_n;
        const int prime = mine ? prime_at(e, a.l, a.L) : 0;
        const Modulus q = modulus(a.fprimes, prime);
        const double* head = a.sfwd + (u64)prime * a.table_stride;
        const rsrc_t dst = make_rsrc((double*)a.out + b * a.out_bs + (u64)(a.dg[digit].out_pos0 + e) * n, (uint32_t)n * 8u);
        double v[NR];
        for (int c0 = 0; c0 < n_src; c0 += chunk) {
            const int c1 = min(c0 + chunk, n_src);
            if (!resident || round == 0) {
                if (c0 || round) __syncthreads();      // every wave is done with the chunk before
                for (int i = c0 + wave; i < c1; i += waves) {
                    const int sp = prime_at(a.src_pos0 + src0 + i, a.l, a.L);
                    const Modulus qs = modulus(a.fprimes, sp);
                    const double* shead = a.sinv + (u64)sp * a.table_stride;
                    double w[NR], last[8] = {};
#pragma unroll
                    for (int r = 0; r < NR; r++)
                        w[r] = bloadf(mid, in_lane, (uint32_t)(i * n * 8u) + (uint32_t)(RB == 5 ? (r >> 1) * 4 + (r & 1) : r) * 8192u);
                    if (RB == 5) {
                        const rsrc_t hr = make_rsrc(shead, HEAD * 8);
#pragma unroll
                        for (int k = 0; k < 4; k++) bload2(hr, (uint32_t)h * 64u, 128u + (uint32_t)k * 16u, last[2 * k], last[2 * k + 1]);
                    }
                    double f = as_const(&a.fprimes[sp].p)[3];                     // N^-1, times the limb's factor
                    if (a.post) f = fp_mulmod(f, as_const(a.post)[src0 + i], qs.p, qs.pinv);
                    const double fw = fp_mulmod(f, as_const(shead)[1], qs.p, qs.pinv);
                    inv_columns<RB>(w, shead, last, f, fw, qs);
                    double* y = ylds + (i - c0) * NR * 64 + lane;
#pragma unroll
                    for (int r = 0; r < NR; r += 2) { y[r * 64] = w[r]; y[r * 64 + 64] = w[r + 1]; }
                }
                __syncthreads();
            }
            if (mine) {
                const cdouble_ptr hat = as_const(a.dg[digit].hat) + prime;
                const double* y0 = ylds + lane;
                if (!HELD || c0 == 0) {
#pragma unroll
                    for (int r = 0; r < NR; r++) v[r] = 0.0;
                }
                if (n_src == 1) {                      // rescale, digits of one limb: the sum's reduction costs more than a product
                    const double f = hat[0];
#pragma unroll
                    for (int r = 0; r < NR; r++) v[r] = fp_norm(fp_mulmod(y0[r * 64], f, q.p, q.pinv), q.p, q.pinv);
                } else {
                    for (int i0 = c0; i0 < c1; i0 += FP_SUM_TERMS) {
                        FpSum s[NR];
#pragma unroll
                        for (int r = 0; r < NR; r++) s[r] = FpSum{FP_SUM_BASE, v[r]};
                        const int i1 = min(i0 + FP_SUM_TERMS, c1);
                        const double* y = y0 + (i0 - c0) * NR * 64;
                        // in pairs: a term leaves its sum in another register, which the end of a loop would copy back
                        int i = i0;
#pragma unroll 1
                        for (; i + 1 < i1; i += 2, y += 2 * NR * 64) {
                            const double f0 = hat[(u64)i * a.total], f1 = hat[(u64)(i + 1) * a.total];
#pragma unroll
                            for (int r = 0; r < NR; r++) {
                                fp_sum_add(s[r], y[r * 64], f0);
                                fp_sum_add(s[r], y[(NR + r) * 64], f1);
                            }
                        }
                        if (i < i1) {
                            const double f0 = hat[(u64)i * a.total];
#pragma unroll
                            for (int r = 0; r < NR; r++) fp_sum_add(s[r], y[r * 64], f0);
                        }
#pragma unroll
                        for (int r = 0; r < NR; r++) v[r] = fp_norm(fp_sum_value(s[r], FP_SUM_BASE, q.p, q.pinv), q.p, q.pinv);
                    }
                }
                if (!HELD || c1 == n_src) {
                    double last[8] = {};
                    if (RB == 5) {
                        const rsrc_t hr = make_rsrc(head, HEAD * 8);
#pragma unroll
                        for (int k = 0; k < 4; k++) bload2(hr, (uint32_t)h * 64u, 128u + (uint32_t)k * 16u, last[2 * k], last[2 * k + 1]);
                    }
                    fwd_columns<RB>(v, head, last, q);
#pragma unroll
                    for (int r = 0; r < NR; r++)
                        bstoref(dst, in_lane, (uint32_t)(RB == 5 ? (r >> 1) * 4 + (r & 1) : r) * 8192u, v[r]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// rows, forward
// ---------------------------------------------------------------------------
template <int K3, int MODE>
__device__ __forceinline__ void rows_forward(const ConvertArgs& a, int n_tasks, double* lds_all) {
    const int task = row_task(n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    double* lds = lds_all + (threadIdx.x >> 6) * ROW_LDS;
    const uint32_t unit = (uint32_t)task / a.n_entries;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const uint32_t row = unit & ((1u << K3) - 1);
    int t = (int)(unit >> K3);
    int digit = 0;
    while (digit + 1 < a.n_digits && t >= a.ext_limbs - a.dg[digit].own_n) { t -= a.ext_limbs - a.dg[digit].own_n; digit++; }
    const int e = t < a.dg[digit].own_lo ? t : t + a.dg[digit].own_n;
    const int prime = prime_at(e, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    u64* out_p = a.out + b * a.out_bs + (u64)(a.dg[digit].out_pos0 + e) * n + row * 1024u;
    const rsrc_t dst = make_rsrc(out_p, 8192u);

    double v[16];
    float m[16];
    load_row(v, dst, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
    RowTwiddles w;
    load_row_twiddles(w, a.sfwd, a.table_stride, prime, row, lane);
    row_forward(v, m, w, lds, lane, q, MODE == FP_FWD_CONV ? BOUND_LIMIT : 5.2f);    // 5.2 p and the accumulator's 2.75 p stay below 8 p

    if (MODE == FP_FWD_CONV) {
        // the extended digits stay doubles: their only readers multiply them by key values in the same arithmetic
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = fp_norm(v[r], q.p, q.pinv);
        store_row(dst, lane, v);
        return;
    }
    double va[16];
    load_row(va, make_rsrc(a.acc + b * a.acc_bs + (u64)e * n + row * 1024u, 8192u), lane);
    if (MODE == FP_FWD_SUB) {      // out = acc - transform: acc already is (sum * P^-1 + addend), the table carries the P^-1
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = va[r] - v[r];
        store_residues(dst, lane, v, q);
        return;
    }
    // out = (acc - transform) * P^-1 (+ addend)
    const double pin = as_const(a.pinv_tab)[prime];
    const bool with_add = a.add && (int)(b % a.add_div) < a.add_polys;
    from_residues(va);
    if (with_add) {
        double vb[16];
        load_row_through<K3>(vb, a.add + (b / a.add_div) * a.add_bs + (b % a.add_div) * a.add_ps + (u64)e * n, 0, row, lane);
        from_residues(vb);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = fp_mulmod(va[r] - v[r], pin, q.p, q.pinv) + vb[r];
    } else {
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = fp_mulmod(va[r] - v[r], pin, q.p, q.pinv);
    }
    store_residues(dst, lane, v, q);
}

// ---------------------------------------------------------------------------
// rows, forward, with the key inner product and the inverse rows of the ModDown's sources
// ---------------------------------------------------------------------------
// One pair of waves per (limb x, row, entry).  The digits' rows are shared out between the two: forward levels (or, for the
// limb's own digit, the input polynomial itself, read through sigma_g), result left in LDS; then wave p multiplies all of
// them by the key's rows of polynomial p.  The sums never leave the registers before they are what the next launch reads:
// limbs below n_acc leave as sum * c1[x] + addend, limbs from n_acc on (the sources of the division that follows)
// go straight through the inverse levels of the row.  A wave that kept both sums beside a row and its twiddles needed 168
// registers and spilled; a pair keeps each wave within 128, four waves per SIMD.
// Per entry the launch reads (digits' limbs) + own + addend and writes 2 (n_acc + sources) limbs: bound by memory.
// Bounds, keys and constants centred: a term is at most 0.501 + 3/16 * 5.5 = 1.54 p, four of them 6.2 p; sum * c1 at most
// 0.501 + 3/16 * 6.2 = 1.7 p; with the addend 2.7 p.
// Several rotations of the same digits (STEPS): the digits come transformed and their rows are read through sigma_g, which maps
// rows to rows; the rest is the same.  The entries of a row, all rotations of it, are neighbours in the order of the tasks, so
// the digits of a limb (the same for all of them) stay in the L2; the keys, each read once, are what the launches stream.
// 24 rotations of one ciphertext at N = 2^14, 12 limbs: 187 -> 162 us against inner products and a division as separate
// launches with the accumulators in memory between them.
// Accesses are 16 bytes a lane: at four waves a SIMD, each waiting for one row at a time, three reads and a write in 8-byte
// accesses run at 4.9 TB/s here and at 5.4 in 16-byte ones (5.3 and 5.4 with all wave slots filled).  64 rotations at N = 2^15, 16 limbs:
// the limbs of q 550 -> 517 us, the special ones 199 -> 190.  Tried and taken back there: two waves a SIMD with everything fetched
// ahead (603 and 235), two entries a workgroup for the sake of the key rows (557), other orders of the tasks (549 .. 556).
#define IP_CAP 5.5f
struct OneStep {};
template <int K3, int MODE, bool ONCE, class S>
__device__ __forceinline__ void rows_inner(const ConvertArgs& a, const InnerArgs& g, const S& s, int n_tasks, double* lds_all) {
    constexpr bool STEPS = !std::is_same<S, OneStep>::value;
    const int per = (n_tasks + 7) >> 3;
    const int task = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (task >= n_tasks) return;
    const int lane = threadIdx.x & 63, at = row_at(lane);
    const int poly = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double* lds = lds_all + poly * ROW_LDS;
    const uint32_t unit = (uint32_t)task / a.n_entries;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const uint32_t row = unit & ((1u << K3) - 1);
    const int x = g.x_end - 1 - (int)(unit >> K3);              // the limbs with the inverse levels, the longest tasks, first
    const int prime = prime_at(x, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    u64 ct = b, galois = g.galois;
    const u64* key = g.key;
    if constexpr (STEPS) {
        const uint32_t step = (uint32_t)b / s.step_B;
        ct = (uint32_t)b - step * s.step_B;
        galois = s.steps.galois[step];
        key = s.steps.key[step];
    }
    double sum[16];
#pragma unroll
    for (int r = 0; r < 16; r++) sum[r] = 0.0;
    for (int d0 = 0; d0 < a.n_digits; d0 += 2) {
        const int d = d0 + poly;
        if (d0) __syncthreads();           // both waves are done with the rows of the two digits before
        if (d < a.n_digits) {
            double v[16];
            if (x >= a.dg[d].own_lo && x < a.dg[d].own_lo + a.dg[d].own_n) {
                load_row_through<K3>(v, g.own + ct * g.own_bs + (u64)x * n, galois, row, lane);
                from_residues(v);
#pragma unroll
                for (int r = 0; r < 16; r++) lds[at + ROW_REG(r)] = v[r];
            } else if (STEPS) {
                load_row_through<K3>(v, a.out + ct * a.out_bs + (u64)(a.dg[d].out_pos0 + x) * n, galois, row, lane);
#pragma unroll
                for (int r = 0; r < 16; r++) lds[at + ROW_REG(r)] = v[r];
            } else {
                const rsrc_t src = make_rsrc((const double*)a.out + b * a.out_bs + (u64)(a.dg[d].out_pos0 + x) * n + row * 1024u, 8192u);
                float m[16];
                load_row(v, src, lane);
#pragma unroll
                for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
                RowTwiddles w;
                row_tables(w, a.sfwd, a.table_stride, prime, row);
                int tl = lane;
                asm volatile("" : "+v"(tl));       // keeps the twiddle loads inside the loop: hoisted they cost 40 registers
                load_twiddles_b(w, tl);
                row_forward<true, true>(v, m, w, lds, tl, q, IP_CAP);
            }
        }
        SCHED_FENCE();
        const double* key_p = (const double*)key + (((u64)d0 * 2 + poly) * a.total + prime) * n + row * 1024u;
        const bool two = d0 + 1 < a.n_digits;
        const rsrc_t k0r = make_rsrc(key_p, 8192u), k1r = make_rsrc(two ? key_p + (u64)2 * a.total * n : key_p, 8192u);
        double k0[16], k1[16];
        load_key_row<ONCE>(k0, k0r, lane);
        // (also without a second digit, then of the first: words left undefined would stay live through the loop)
        load_key_row<ONCE>(k1, k1r, lane);
        SCHED_FENCE();
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; r++) sum[r] += fp_mulmod(lds_all[at + ROW_REG(r)], k0[r], q.p, q.pinv);
        if (two) {
#pragma unroll
            for (int r = 0; r < 16; r++) sum[r] += fp_mulmod(lds_all[ROW_LDS + at + ROW_REG(r)], k1[r], q.p, q.pinv);
        }
        if (d0 % 4 == 2 && d0 + 2 < a.n_digits) {
#pragma unroll
            for (int r = 0; r < 16; r++) sum[r] = fp_norm(sum[r], q.p, q.pinv);
        }
    }
    const double c1 = as_const(g.c1)[x];
    const bool source = MODE == FP_INV_D_TO_Y && x >= g.n_acc;
#pragma unroll
    for (int r = 0; r < 16; r++) sum[r] = fp_mulmod(sum[r], c1, q.p, q.pinv);
    SCHED_FENCE();
    if (x < a.l && poly < g.add_polys) {
        double t[16];
        load_row_through<K3>(t, g.add + ct * g.add_bs + (u64)poly * g.add_ps + (u64)x * n, galois, row, lane);
        from_residues(t);
        if (g.c2) {
            const double c2 = as_const(g.c2)[x];
#pragma unroll
            for (int r = 0; r < 16; r++) t[r] = fp_mulmod(t[r], c2, q.p, q.pinv);
        }
#pragma unroll
        for (int r = 0; r < 16; r++) sum[r] += t[r];
    }
    SCHED_FENCE();
    const u64 out_limb = source ? (b * 2 + poly) * (u64)(a.ext_limbs - g.n_acc) + (u64)(x - g.n_acc) : (b * 2 + poly) * (u64)g.n_acc + (u64)x;
    double* dst_p = (source ? g.down : MODE == FP_FWD_CONV_SUB ? (double*)g.out : g.acc) + out_limb * n + row * 1024u;
    const rsrc_t dst = make_rsrc(dst_p, 8192u);
    if (source) {
        __syncthreads();                   // uniform in the workgroup: the other wave still reads this one's row
        float m[16];
#pragma unroll
        for (int r = 0; r < 16; r++) m[r] = 2.75f;
        RowTwiddles w;
        load_row_twiddles(w, a.sinv, a.table_stride, prime, row, lane);
        row_inverse(sum, m, w, lds, lane, q);
    } else if (MODE == FP_FWD_CONV_SUB) {  // the division's columns are there already: its rows, and the difference
        double v[16];
        float m[16];
        load_row(v, dst, lane);
#pragma unroll
        for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
        RowTwiddles w;
        load_row_twiddles(w, a.sfwd, a.table_stride, prime, row, lane);
        __syncthreads();
        row_forward(v, m, w, lds, lane, q, 5.2f);
#pragma unroll
        for (int r = 0; r < 16; r++) v[r] = sum[r] - v[r];
        store_residues(dst, lane, v, q);
        return;
    }
    store_row(dst, lane, sum);
}

// ---------------------------------------------------------------------------
// rows by four waves each: calls with few rows
// ---------------------------------------------------------------------------
#define WIDE_DIGITS 4    // at most, in an inner product: four waves each
struct WideTwiddles { double w[5][3]; };     // per stage: level 2 s, then the two groups of level 2 s + 1
// (t: thread of the row; tables as split_table_words lays them out)
__device__ __forceinline__ void wide_twiddles(WideTwiddles& w, const double* table, u64 stride, int prime, uint32_t row, uint32_t t, Modulus q) {
    const double* head = table + (u64)prime * stride;
    const double* tab = head + HEAD + (u64)row * SPLIT_ROW;
    const rsrc_t tr = make_rsrc(tab, SPLIT_ROW * 8), hr = make_rsrc(head + 32, 16 * 8);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    const uint32_t g = t >> 4, b = t >> 3, k = t & 7, odd = (t >> 2) & 1;
    w.w[2][0] = bloadf(tr, ((g & 1) * 8 + (g >> 1)) * 8u, 16 * 8);
    bload2(tr, g * 16u, 32 * 8, w.w[2][1], w.w[2][2]);
    const double c1 = bloadf(tr, b * 8u, 64 * 8), c2 = bloadf(tr, b * 8u, 96 * 8), c3 = bloadf(tr, b * 8u, 128 * 8);
    const double f1 = bloadf(hr, odd * 8u, 0), f3 = bloadf(hr, k * 8u, 0);
    double f20, f21;
    bload2(hr, odd * 16u, 0, f20, f21);
    const uint32_t last = ((k >> 1) * 128 + b * 2 + (k & 1)) * 8u;
    w.w[4][1] = bloadf(tr, last, 160 * 8);
    w.w[4][2] = bloadf(tr, last, 160 * 8 + 512);
    w.w[0][0] = as_const(tab)[1]; w.w[0][1] = as_const(tab)[2]; w.w[0][2] = as_const(tab)[3];
    w.w[1][0] = as_const(tab)[4 + wave]; w.w[1][1] = as_const(tab)[8 + 2 * wave]; w.w[1][2] = as_const(tab)[9 + 2 * wave];
    w.w[3][0] = fp_mulmod(c1, f1, q.p, q.pinv);
    w.w[3][1] = fp_mulmod(c2, f20, q.p, q.pinv);
    w.w[3][2] = fp_mulmod(c2, f21, q.p, q.pinv);
    w.w[4][0] = fp_mulmod(c3, f3, q.p, q.pinv);
}
__device__ __forceinline__ void wide_cap(double (&v)[4], float (&m)[4], float cap, Modulus q) {
#pragma unroll
    for (int r = 0; r < 4; r++)
        if (m[r] > cap) v[r] = fp_norm(v[r], q.p, q.pinv);
}
// bounds of the twiddles: tables up to stage 2, products behind
#define WIDE_TW_BOUND(s) (s < 3 ? 0.5f : 0.6f)
// in: below `bound` p; out: below cap p
__device__ __forceinline__ void wide_forward(double (&v)[4], float bound, const WideTwiddles& w, double* lds, uint32_t t, Modulus q, float cap) {
    float m[4] = {bound, bound, bound, bound};
    wide_forward_levels(v, m, lds, t, [&](auto s, double& x, double& y, float& bx, float& by, int k) {
        fwd_bfly(x, y, bx, by, w.w[s][k], WIDE_TW_BOUND(s), q);
    });
    wide_cap(v, m, cap, q);
}
// in: below `bound` p; out: below 1.01 p
__device__ __forceinline__ void wide_inverse(double (&v)[4], float bound, const WideTwiddles& w, double* lds, uint32_t t, Modulus q) {
    float m[4] = {bound, bound, bound, bound};
    wide_inverse_levels(v, m, lds, t, [&](auto s, double& x, double& y, float& bx, float& by, int k) {
        inv_bfly(x, y, bx, by, w.w[s][k], WIDE_TW_BOUND(s), q);
    });
    wide_cap(v, m, 1.01f, q);
}
__device__ __forceinline__ void wide_from_residues(double (&v)[4]) {
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = fp_from_u64((u64)__double_as_longlong(v[r]));
}
__device__ __forceinline__ void wide_store_residues(rsrc_t dst, uint32_t t, double (&v)[4], Modulus q) {
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = __longlong_as_double((long long)fp_canonical(v[r], q.p, q.pinv));
    wide_store(dst, t, v);
}

template <int K3>
__device__ __forceinline__ void wide_rows_inverse(const ConvertArgs& a, int task, double* lds) {
    const uint32_t t = threadIdx.x, unit = (uint32_t)task / a.n_entries, b = (uint32_t)task - unit * a.n_entries;
    const uint32_t row = unit & ((1u << K3) - 1), k = unit >> K3;
    const int prime = prime_at(a.src_pos0 + (int)k, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    double v[4];
    WideTwiddles w;
    wide_load<K3>(v, a.in + (u64)b * a.in_bs + (u64)(a.src_pos0 + (int)k) * n, a.galois, row, t);
    wide_twiddles(w, a.sinv, a.table_stride, prime, row, t, q);
    wide_from_residues(v);
    wide_inverse(v, 1.0f, w, lds, t, q);
    const rsrc_t dst = make_rsrc(a.mid + ((u64)b * a.n_src + k) * n + row * 1024u, 8192u);
#pragma unroll
    for (int r = 0; r < 4; r++) bstoref(dst, t * 8u, (uint32_t)r * 2048u, v[r]);
}

template <int K3, int MODE>
__device__ __forceinline__ void wide_rows_forward(const ConvertArgs& a, int task, double* lds) {
    const uint32_t t = threadIdx.x, unit = (uint32_t)task / a.n_entries;
    const u64 b = (uint32_t)task - unit * a.n_entries;
    const uint32_t row = unit & ((1u << K3) - 1);
    int e = (int)(unit >> K3), digit = 0;
    while (digit + 1 < a.n_digits && e >= a.ext_limbs - a.dg[digit].own_n) { e -= a.ext_limbs - a.dg[digit].own_n; digit++; }
    if (e >= a.dg[digit].own_lo) e += a.dg[digit].own_n;
    const int prime = prime_at(e, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)(a.dg[digit].out_pos0 + e) * n + row * 1024u, 8192u);
    double v[4], acc[4], add[4];
    WideTwiddles w;
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = bloadf(dst, t * 8u, (uint32_t)r * 2048u);
    wide_twiddles(w, a.sfwd, a.table_stride, prime, row, t, q);
    const bool with_add = MODE == FP_FWD_CONV_FINAL && a.add && (int)(b % a.add_div) < a.add_polys;
    if (MODE != FP_FWD_CONV) wide_load<K3>(acc, a.acc + b * a.acc_bs + (u64)e * n, 0, row, t);
    if (with_add) wide_load<K3>(add, a.add + (b / a.add_div) * a.add_bs + (b % a.add_div) * a.add_ps + (u64)e * n, 0, row, t);
    wide_forward(v, COLUMNS_BOUND, w, lds, t, q, MODE == FP_FWD_CONV ? BOUND_LIMIT : 5.2f);
    if (MODE == FP_FWD_CONV) {
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = fp_norm(v[r], q.p, q.pinv);
        wide_store(dst, t, v);
        return;
    }
    if (MODE == FP_FWD_SUB) {
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = acc[r] - v[r];
    } else {
        const double pin = as_const(a.pinv_tab)[prime];
        wide_from_residues(acc);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = fp_mulmod(acc[r] - v[r], pin, q.p, q.pinv);
        if (with_add) {
            wide_from_residues(add);
#pragma unroll
            for (int r = 0; r < 4; r++) v[r] += add[r];
        }
    }
    wide_store_residues(dst, t, v, q);
}

// A workgroup per (limb x, row, entry), four waves per digit.  Each four leave their digit's row in LDS; the first two take a
// polynomial each from there on: sums, and the inverse rows of a source or the division's rows, as rows_inner does.  split: a workgroup
// per polynomial too, for launches that leave compute units idle (the rule stands at the launch): the digits' rows are transformed for
// either, and what follows them is left to four waves that have waited with keys and twiddles in registers (with four digits, to those of
// the first).
template <int K3, int MODE>
__device__ __forceinline__ void wide_rows_inner(const ConvertArgs& a, const InnerArgs& g, int task, double* lds) {
    const uint32_t t = threadIdx.x & (WIDE_NT - 1);
    const int part = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WIDE_NT));
    const uint32_t entry = (uint32_t)task >> g.split, unit = entry / a.n_entries;
    const u64 b = entry - unit * a.n_entries;
    const int summer = a.n_digits < WIDE_DIGITS ? a.n_digits : 0, poly = g.split ? task & 1 : part;
    const uint32_t row = unit & ((1u << K3) - 1);
    const int x = g.x_end - 1 - (int)(unit >> K3);
    const int prime = prime_at(x, a.l, a.L);
    const Modulus q = modulus(a.fprimes, prime);
    constexpr u64 n = (u64)1 << (10 + K3);
    const bool sums = g.split ? part == summer : part < 2, source = MODE == FP_INV_D_TO_Y && x >= g.n_acc, mine = part < a.n_digits;
    const bool own = mine && x >= a.dg[part].own_lo && x < a.dg[part].own_lo + a.dg[part].own_n;
    const bool with_add = sums && x < a.l && poly < g.add_polys;
    const u64 out_limb = source ? (b * 2 + poly) * (u64)(a.ext_limbs - g.n_acc) + (u64)(x - g.n_acc) : (b * 2 + poly) * (u64)g.n_acc + (u64)x;
    double* dst_p = (source ? g.down : MODE == FP_FWD_CONV_SUB ? (double*)g.out : g.acc) + (sums ? out_limb : 0) * n + row * 1024u;
    const rsrc_t dst = make_rsrc(dst_p, 8192u);
    double v[4], k[WIDE_DIGITS][4], add[4], div[4];
    WideTwiddles w;
    double* slot = lds + part * WIDE_LDS;
    if (own) {
        wide_load<K3>(v, g.own + b * g.own_bs + (u64)x * n, g.galois, row, t);
    } else if (mine) {
        const rsrc_t src = make_rsrc((const double*)a.out + b * a.out_bs + (u64)(a.dg[part].out_pos0 + x) * n + row * 1024u, 8192u);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = bloadf(src, t * 8u, (uint32_t)r * 2048u);
    }
    const bool waits = sums && !mine;                            // has no digit
    if (waits && source) wide_twiddles(w, a.sinv, a.table_stride, prime, row, t, q);
    else if (!own || MODE == FP_FWD_CONV_SUB) wide_twiddles(w, a.sfwd, a.table_stride, prime, row, t, q);
    if (sums) {
#pragma unroll
        for (int d = 0; d < WIDE_DIGITS; d++)
            if (d < a.n_digits) wide_load<K3>(k[d], g.key + (((u64)d * 2 + poly) * a.total + prime) * n, 0, row, t);
        if (with_add) wide_load<K3>(add, g.add + b * g.add_bs + (u64)poly * g.add_ps + (u64)x * n, g.galois, row, t);
        if (MODE == FP_FWD_CONV_SUB) {
#pragma unroll
            for (int r = 0; r < 4; r++) div[r] = bloadf(dst, t * 8u, (uint32_t)r * 2048u);
        }
    }
    if (mine && !own) wide_forward(v, COLUMNS_BOUND, w, slot, t, q, IP_CAP);
    else wide_no_row();
    if (own) wide_from_residues(v);
    if (mine) {
#pragma unroll
        for (int r = 0; r < 4; r++) slot[wide_at(4 * t + r)] = v[r];
    }
    if (sums && source && !waits) wide_twiddles(w, a.sinv, a.table_stride, prime, row, t, q);      // on their way while the sums are formed
    __syncthreads();
    if (sums) {
        const double c1 = as_const(g.c1)[x];
#pragma unroll
        for (int r = 0; r < 4; r++) {
            double sum = 0.0;
#pragma unroll
            for (int d = 0; d < WIDE_DIGITS; d++)
                if (d < a.n_digits) sum += fp_mulmod(lds[d * WIDE_LDS + wide_at(4 * t + r)], k[d][r], q.p, q.pinv);
            v[r] = fp_mulmod(sum, c1, q.p, q.pinv);
        }
        if (with_add) {
            wide_from_residues(add);
            const double c2 = g.c2 ? as_const(g.c2)[x] : 1.0;
#pragma unroll
            for (int r = 0; r < 4; r++) v[r] += fp_mulmod(add[r], c2, q.p, q.pinv);
        }
        if (!source && MODE == FP_INV_D_TO_Y) wide_store(dst, t, v);
    }
    if (!source && MODE == FP_INV_D_TO_Y) return;
    __syncthreads();                                            // everyone has read the digits
    if (!sums) {
        wide_no_row();
        return;
    }
    if (MODE == FP_FWD_CONV_SUB) {
        wide_forward(div, COLUMNS_BOUND, w, slot, t, q, 5.2f);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] -= div[r];
        wide_store_residues(dst, t, v, q);
    } else {
        wide_inverse(v, 2.75f, w, slot, t, q);
#pragma unroll
        for (int r = 0; r < 4; r++) bstoref(dst, t * 8u, (uint32_t)r * 2048u, v[r]);
    }
}

// ---------------------------------------------------------------------------
// whole polynomials by columns and rows: calls with few of them (encode, decode, encryption of a few vectors)
// ---------------------------------------------------------------------------
// The single-launch transform of ntt_fp.hip reads and writes a polynomial once but takes 13 / 20 / 35 us at N = 2^13 / 14 /
// 15 however few there are; this form moves it twice and takes about 5 us a launch until the chip is full.
// Tasks are waves, (limb, entry, tile of columns) or (limb, entry, row).

__device__ __forceinline__ double residue_of_i64(i64 v, Modulus q) {     // any 64-bit integer, as a normalised double
    const double hi = (double)(v >> 30), lo = (double)(v & 0x3fffffff);  // |hi| <= 2^33
    return fp_norm(fp_mulmod(hi, 1073741824.0, q.p, q.pinv) + lo, q.p, q.pinv);
}

template <int K3>
__device__ __forceinline__ void load_last(double (&last)[8], const double* head, int h) {
    if (K3 != 5) return;
    const rsrc_t hr = make_rsrc(head, HEAD * 8);
#pragma unroll
    for (int k = 0; k < 4; k++) bload2(hr, (uint32_t)h * 64u, 128u + (uint32_t)k * 16u, last[2 * k], last[2 * k + 1]);
}

// byte offset of register r's row before the forward / after the inverse levels on `a` (FIRST), and on the other side
template <int K3, bool FIRST>
__device__ __forceinline__ uint32_t column_row(int r) { return (uint32_t)(K3 != 5 ? r : FIRST ? 2 * r : (r >> 1) * 4 + (r & 1)) * 8192u; }
template <int K3, bool FIRST>
__device__ __forceinline__ uint32_t column_lane(int tile, int lane) {
    return (uint32_t)(K3 != 5 ? tile * 64 + lane : tile * 32 + (lane & 31) + (lane >> 5) * (FIRST ? 1024 : 2048)) * 8u;
}

template <int K3, bool INV>
__device__ __forceinline__ void plain_columns(const FpArgs& a, const FpTask& tk) {
    constexpr int NR = Col<K3>::NR, TILES = 1024 / Col<K3>::WIDTH;
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = row_task(a.n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63, tile = task & (TILES - 1), unit = task / TILES;
    const int e = unit / a.n_entries;
    const u64 b = unit - e * a.n_entries;
    const int prime = tk.prime[e];
    const Modulus q = modulus(a.fprimes, prime);
    const double* head = (INV ? a.sinv : a.sfwd) + (u64)prime * a.table_stride;
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)tk.pos[e] * n, (uint32_t)n * 8u);
    const uint32_t first = column_lane<K3, true>(tile, lane), other = column_lane<K3, false>(tile, lane);
    double v[NR], last[8] = {};
    load_last<K3>(last, head, lane >> 5);
    if (INV) {
#pragma unroll
        for (int r = 0; r < NR; r++) v[r] = bloadf(dst, other, column_row<K3, false>(r));
        const double f = as_const(&a.fprimes[prime].p)[3], fw = fp_mulmod(f, as_const(head)[1], q.p, q.pinv);
        inv_columns<K3>(v, head, last, f, fw, q);
#pragma unroll
        for (int r = 0; r < NR; r++) {
            if (a.centred_out) bstoref(dst, first, column_row<K3, true>(r), v[r]);
            else bstore(dst, first, column_row<K3, true>(r), fp_to_u64(v[r] < 0.0 ? v[r] + q.p : v[r]));
        }
    } else {
        if (a.coeffs) {
            const rsrc_t src = make_rsrc(a.coeffs + b * n, (uint32_t)n * 8u);
            u64 c[NR];
#pragma unroll
            for (int r = 0; r < NR; r++) c[r] = bload(src, first, column_row<K3, true>(r));
#pragma unroll
            for (int r = 0; r < NR; r++) v[r] = residue_of_i64((i64)c[r], q);
        } else {
            const rsrc_t src = make_rsrc(a.in + b * a.in_bs + (u64)tk.pos[e] * n, (uint32_t)n * 8u);
            u64 c[NR];
#pragma unroll
            for (int r = 0; r < NR; r++) c[r] = bload(src, first, column_row<K3, true>(r));
#pragma unroll
            for (int r = 0; r < NR; r++) v[r] = fp_norm(fp_from_u64(c[r]), q.p, q.pinv);
        }
        fwd_columns<K3>(v, head, last, q);
#pragma unroll
        for (int r = 0; r < NR; r++) bstoref(dst, other, column_row<K3, false>(r), v[r]);
    }
}

template <int K3, bool INV>
__device__ __forceinline__ void plain_rows(const FpArgs& a, const FpTask& tk, double* lds_all) {
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = row_task(a.n_tasks);
    if (task < 0) return;
    const int lane = threadIdx.x & 63, row = task & ((1 << K3) - 1), unit = task >> K3;
    double* lds = lds_all + (threadIdx.x >> 6) * ROW_LDS;
    const int e = unit / a.n_entries;
    const u64 b = unit - e * a.n_entries;
    const int prime = tk.prime[e];
    const Modulus q = modulus(a.fprimes, prime);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)tk.pos[e] * n + (u64)row * 1024u, 8192u);
    double v[16];
    float m[16];
    RowTwiddles w;
    if (INV) {
        load_row_through<K3>(v, a.in + b * a.in_bs + (u64)tk.pos[e] * n, 0, (uint32_t)row, lane);
        load_row_twiddles(w, a.sinv, a.table_stride, prime, (uint32_t)row, lane);
        from_residues(v);
#pragma unroll
        for (int r = 0; r < 16; r++) m[r] = 1.0f;
        row_inverse(v, m, w, lds, lane, q);
        store_row(dst, lane, v);
    } else {
        load_row(v, dst, lane);
#pragma unroll
        for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
        load_row_twiddles(w, a.sfwd, a.table_stride, prime, (uint32_t)row, lane);
        row_forward(v, m, w, lds, lane, q, BOUND_LIMIT);
        store_residues(dst, lane, v, q);
    }
}

// the same by four waves a row
template <int K3, int MODE>
__global__ __launch_bounds__(WIDE_NT, 4) void ntt_fp_split_wide_kernel(FpArgs a, FpTask tk) {
    __shared__ double lds[WIDE_LDS];
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = wide_task(a.n_tasks);
    if (task < 0) return;
    const uint32_t t = threadIdx.x, row = (uint32_t)task & ((1u << K3) - 1);
    const int unit = task >> K3, e = unit / a.n_entries;
    const u64 b = unit - e * a.n_entries;
    const int prime = tk.prime[e];
    const Modulus q = modulus(a.fprimes, prime);
    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)tk.pos[e] * n + (u64)row * 1024u, 8192u);
    double v[4];
    WideTwiddles w;
    if (MODE == FP_INV_PLAIN) {
        wide_load<K3>(v, a.in + b * a.in_bs + (u64)tk.pos[e] * n, 0, row, t);
        wide_twiddles(w, a.sinv, a.table_stride, prime, row, t, q);
        wide_from_residues(v);
        wide_inverse(v, 1.0f, w, lds, t, q);
#pragma unroll
        for (int r = 0; r < 4; r++) bstoref(dst, t * 8u, (uint32_t)r * 2048u, v[r]);
    } else {
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] = bloadf(dst, t * 8u, (uint32_t)r * 2048u);
        wide_twiddles(w, a.sfwd, a.table_stride, prime, row, t, q);
        wide_forward(v, COLUMNS_BOUND, w, lds, t, q, BOUND_LIMIT);
        wide_store_residues(dst, t, v, q);
    }
}

template <int K3, int MODE, bool COLUMNS>
__global__ __launch_bounds__(ROWS_NT, 4) void ntt_fp_split_kernel(FpArgs a, FpTask tk) {
    if constexpr (COLUMNS) {
        plain_columns<K3, MODE == FP_INV_PLAIN>(a, tk);
    } else {
        __shared__ double lds[4 * ROW_LDS];
        plain_rows<K3, MODE == FP_INV_PLAIN>(a, tk, lds);
    }
}

// Encryption of a batch: the columns launch draws the uniform polynomial a (into polynomial 1 of the ciphertexts) and the
// error e (polynomial 0) while it loads them, the rows launch finishes both transforms of a row and stores (-a s + e + m, a).
// Few vectors are bound by the chain of a wave: the table of e fetched anew for each of sixteen samples was most of it (4 vectors
// at N = 2^14, 12 limbs, 23.5 us against 14.8 with an entry serving all of them).  The samples held for that take registers -- five waves a
// SIMD instead of eight at N = 2^14, four instead of six at 2^15 -- and it is ahead all the same for many: both launches, us, 1, 4, 16 and 64
// vectors at N = 2^14, 12 limbs 22.8, 29.1, 56.6, 166 -> 12.3, 19.6, 45.2, 148; at 2^15, 21 limbs 29, 56, 157, 620 -> 19, 42, 136, 565.
template <int K3>
__global__ __launch_bounds__(ROWS_NT, 4) void encrypt_columns_kernel(EncryptArgs a) {
    constexpr int NR = Col<K3>::NR, TILES = 1024 / Col<K3>::WIDTH;
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = row_task(a.n_entries * a.limbs * 2 * TILES);
    if (task < 0) return;
    const int lane = threadIdx.x & 63, tile = task & (TILES - 1), unit = task / TILES;
    const int poly = unit & 1, limb = (unit >> 1) / a.n_entries;
    const u64 b = (unit >> 1) - limb * a.n_entries;
    const Modulus q = modulus(a.fprimes, limb);
    const double* head = a.sfwd + (u64)limb * a.table_stride;
    const uint32_t first = column_lane<K3, true>(tile, lane);
    double v[NR], last[8] = {};
    load_last<K3>(last, head, lane >> 5);
    const u64 key = stream_key(a.seed, poly ? 2 : 3, a.ctr + b);
    if (poly) {
        const PrimeConst pc = a.primes[limb];
#pragma unroll
        for (int r = 0; r < NR; r++) {
            const u64 j = (first + column_row<K3, true>(r)) >> 3;
            v[r] = fp_norm(fp_from_u64(barrett128(0, rnd_at(key, (u64)limb * n + j), pc.q, pc.r1, pc.r0)), q.p, q.pinv);
        }
    } else {
        u64 words[NR];
#pragma unroll
        for (int r = 0; r < NR; r++) words[r] = rnd_at(key, (first + column_row<K3, true>(r)) >> 3);
        gaussians_from_words(v, words, a.cdt, a.noise_on ? a.cdt_n : 0);
    }
    fwd_columns<K3>(v, head, last, q);
    const rsrc_t dst = make_rsrc(a.ct + ((b * 2 + poly) * a.limbs + limb) * n, (uint32_t)n * 8u);
    const uint32_t other = column_lane<K3, false>(tile, lane);
#pragma unroll
    for (int r = 0; r < NR; r++) bstoref(dst, other, column_row<K3, false>(r), v[r]);
}

// Two transforms of a row and its products, bound by memory in large batches.  Twiddles fetched per transform, those of c behind the
// levels on b: without spills, us a batch, 8 registers spilled -> none: 64 vectors at N = 2^14, 12 limbs 158.3 -> 156, at N = 2^15, 16
// limbs 467 -> 458; 20 at N = 2^14 68.5 -> 67.2.
template <int K3>
__global__ __launch_bounds__(ROWS_NT, 4) void encrypt_rows_kernel(EncryptArgs a) {
    __shared__ double lds_all[4 * ROW_LDS];
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = row_task((a.n_entries * a.limbs) << K3);
    if (task < 0) return;
    const int lane = threadIdx.x & 63;
    double* lds = lds_all + (threadIdx.x >> 6) * ROW_LDS;
    const int unit = task / a.n_entries;
    const u64 b = task - unit * a.n_entries;
    const int row = unit & ((1 << K3) - 1), limb = unit >> K3;
    const Modulus q = modulus(a.fprimes, limb);
    u64* c0 = a.ct + ((b * 2) * a.limbs + limb) * n + (u64)row * 1024u;
    const rsrc_t r0 = make_rsrc(c0, 8192u), r1 = make_rsrc(c0 + a.limbs * n, 8192u);
    const rsrc_t sk = make_rsrc(a.secret + limb * n + (u64)row * 1024u, 8192u), pt = make_rsrc(a.pt[b] + limb * n + (u64)row * 1024u, 8192u);
    double e[16], v[16], s[16];
    float m[16];
    RowTwiddles w;
    row_tables(w, a.sfwd, a.table_stride, limb, (uint32_t)row);
    load_twiddles_b(w, lane);
    load_row(e, r0, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
    row_forward<true>(e, m, w, lds, lane, q, 3.0f);       // 3 + 1 (message) + 2.5 (a s, below) stays within 8 p
    load_row(v, r1, lane);
#pragma unroll
    for (int r = 0; r < 16; r++) m[r] = COLUMNS_BOUND;
    int tl = lane;
    asm volatile("" : "+v"(tl));           // the twiddles are fetched again: kept beside two rows they spilled
    load_twiddles_b(w, tl);
    row_forward<true>(v, m, w, lds, tl, q, 5.2f);
    load_row(s, sk, lane);
    from_residues(s);
#pragma unroll
    for (int r = 0; r < 16; r++) e[r] -= fp_mulmod(v[r], s[r], q.p, q.pinv);
    store_residues(r1, lane, v, q);
    SCHED_FENCE();
    load_row(s, pt, lane);
    from_residues(s);
#pragma unroll
    for (int r = 0; r < 16; r++) e[r] += s[r];
    store_residues(r0, lane, e, q);
}

// the same by four waves a row, the two transforms side by side
template <int K3>
__global__ __launch_bounds__(2 * WIDE_NT, 4) void encrypt_rows_wide_kernel(EncryptArgs a) {
    __shared__ double lds[2 * WIDE_LDS];
    constexpr u64 n = (u64)1 << (10 + K3);
    const int task = wide_task((a.n_entries * a.limbs) << K3);
    if (task < 0) return;
    const uint32_t t = threadIdx.x & (WIDE_NT - 1);
    const int poly = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WIDE_NT));
    const int unit = task / a.n_entries;
    const u64 b = task - unit * a.n_entries;
    const uint32_t row = (uint32_t)unit & ((1u << K3) - 1);
    const int limb = unit >> K3;
    const Modulus q = modulus(a.fprimes, limb);
    const rsrc_t dst = make_rsrc(a.ct + ((b * 2 + poly) * a.limbs + limb) * n + (u64)row * 1024u, 8192u);
    double v[4], s[4], m[4];
    WideTwiddles w;
    double* slot = lds + poly * WIDE_LDS;
#pragma unroll
    for (int r = 0; r < 4; r++) v[r] = bloadf(dst, t * 8u, (uint32_t)r * 2048u);
    wide_twiddles(w, a.sfwd, a.table_stride, limb, row, t, q);
    if (poly == 0) {
        wide_load<K3>(s, a.secret + limb * n, 0, row, t);
        wide_load<K3>(m, a.pt[b] + limb * n, 0, row, t);
    }
    wide_forward(v, COLUMNS_BOUND, w, slot, t, q, poly ? 5.2f : 3.0f);       // 3 + 1 (message) + 2.5 (a s) stays within 8 p
    if (poly) {
#pragma unroll
        for (int r = 0; r < 4; r++) slot[wide_at(4 * t + r)] = v[r];
    }
    __syncthreads();
    if (poly == 0) {
        wide_from_residues(s);
        wide_from_residues(m);
#pragma unroll
        for (int r = 0; r < 4; r++) v[r] += m[r] - fp_mulmod(lds[WIDE_LDS + wide_at(4 * t + r)], s[r], q.p, q.pinv);
    }
    wide_store_residues(dst, t, v, q);
}

// ---------------------------------------------------------------------------
// the kernel family and its launches
// ---------------------------------------------------------------------------
// MODE (enum FpMode) names the stage a launch belongs to, so that a profile tells the ModUp's columns from the ModDown's;
// COLUMNS: the launch in which all target limbs of a digit share one pass over its sources, else the rows.
constexpr int fp_threads(int mode, bool columns) { return columns ? 1024 : (mode == FP_INV_D_TO_Y || mode == FP_FWD_CONV_SUB) ? 128 : ROWS_NT; }
// waves per SIMD to leave room for: three workgroups of eight waves of the columns at N = 2^15 and 2^14, four at 2^13
constexpr int fp_waves(int k3, bool columns) { return !columns ? 4 : k3 >= 4 ? 6 : k3 == 3 ? 8 : 4; }

template <int K3, int MODE, bool COLUMNS>
__global__ __launch_bounds__(fp_threads(MODE, COLUMNS), fp_waves(K3, COLUMNS)) void ntt_fp_kernel(ConvertArgs a, InnerArgs g, int n_tasks) {
    if constexpr (COLUMNS) {
        extern __shared__ double ylds[];
        columns<K3, false>(a, ylds);
    } else {
        __shared__ double lds[fp_threads(MODE, false) / 64 * ROW_LDS];
        if constexpr (MODE == FP_INV_TO_Y) rows_inverse<K3>(a, n_tasks, lds);
        else if constexpr (MODE == FP_INV_D_TO_Y || MODE == FP_FWD_CONV_SUB) rows_inner<K3, MODE, false>(a, g, OneStep{}, n_tasks, lds);
        else rows_forward<K3, MODE>(a, n_tasks, lds);
    }
}

// columns of digits with more sources than the LDS holds
template <int K3, int MODE>
__global__ __launch_bounds__(1024, 4) void ntt_fp_chunks_kernel(ConvertArgs a) {
    extern __shared__ double ylds[];
    columns<K3, true>(a, ylds);
}

constexpr bool fp_inner(int mode) { return mode == FP_INV_D_TO_Y || mode == FP_FWD_CONV_SUB; }
template <int K3, int MODE>
__global__ __launch_bounds__(fp_inner(MODE) ? WIDE_DIGITS * WIDE_NT : WIDE_NT, 4) void ntt_fp_wide_kernel(ConvertArgs a, InnerArgs g, int n_tasks) {
    extern __shared__ double wide_lds[];
    const int task = wide_task(n_tasks);
    if (task < 0) return;
    if constexpr (MODE == FP_INV_TO_Y) wide_rows_inverse<K3>(a, task, wide_lds);
    else if constexpr (fp_inner(MODE)) wide_rows_inner<K3, MODE>(a, g, task, wide_lds);
    else wide_rows_forward<K3, MODE>(a, task, wide_lds);
}

// the inner products' rows for several rotations of the same digits; ONCE: the keys pass the caches by
template <int K3, int MODE, bool ONCE>
__global__ __launch_bounds__(128, 4) void inner_product_steps_rows_kernel(ConvertArgs a, InnerArgs g, StepArgs s, int n_tasks) {
    __shared__ double lds[2 * ROW_LDS];
    rows_inner<K3, MODE, ONCE>(a, g, s, n_tasks, lds);
}

// Twiddles of one prime for the three kernels, psi^(sign bitrev(i)) as the caller's w(i) gives them (centred doubles):
//   [0 .. 31]   column levels: entry 2^j + g; N = 2^15: the 16 of level 4 as [half h][k], group 2 k + h
//   [32 .. 47]  w(g), g < 16: the factors that turn a thread's twiddle of group 0 into that of group g
//   then per row a, SPLIT_ROW entries (R = N / 1024):
//   [0 .. 31]   levels on b: entry 2^j + g = w(((R + a) 2^j) + g), level 4 as [h][k]
//   [32 .. 159] levels on c, j < 4: [j][b] = w((32 (R + a) + b) 2^j)
//   [160 ..]    level 4 on c: [k / 2][h][b][k & 1] = w(16 (32 (R + a) + b) + 2 k + h)
size_t split_table_words(int log_n) { return HEAD + ((size_t)SPLIT_ROW << (log_n - 10)); }

// every pointer a launch dereferences is set and every limb it names has a prime: a mistake is a host error
static bool convert_args_ok(const ConvertArgs& a, u64* targets) {
    if (a.log_n < 12 || a.log_n > 15 || a.n_digits < 1 || a.n_digits > FP_MAX_DIGITS) return false;
    if (!a.fprimes || !a.sfwd || !a.sinv || !a.mid || !a.out || a.n_src < 1 || a.l < 1 || a.L < a.l || a.total < 1) return false;
    if (a.src_pos0 < 0 || a.ext_limbs < 1) return false;
    auto prime_of = [&](int pos) { return pos < a.l ? pos : pos + (a.L - a.l); };
    if (prime_of(a.src_pos0 + a.n_src - 1) >= a.total || prime_of(a.ext_limbs - 1) >= a.total) return false;
    *targets = 0;
    for (int d = 0; d < a.n_digits; d++) {
        const ConvertArgs::Digit& g = a.dg[d];
        if (!g.hat || g.a < 1 || g.src0 < 0 || g.src0 + g.a > a.n_src || g.own_n < 0 || g.own_lo < 0 || g.own_lo + g.own_n > a.ext_limbs ||
            g.out_pos0 < 0)
            return false;
        *targets += (u64)(a.ext_limbs - g.own_n);
    }
    return (((u64)a.n_src * a.n_entries) << (a.log_n - 10)) <= 0x7fffff00u && ((*targets * a.n_entries) << (a.log_n - 10)) <= 0x7fffff00u;
}

template <int K3, int MODE, bool COLUMNS>
static hipError_t launch_one(dim3 grid, unsigned threads, size_t lds, const ConvertArgs& a, const InnerArgs& g, u64 tasks, hipStream_t st) {
    static char name[40] = "";      // what rocprofv3 prints for this instantiation
    if (!name[0]) snprintf(name, sizeof name, "ntt_fp_kernel<%d, %d, %s>", K3, MODE, COLUMNS ? "true" : "false");
    ProfScope prof__(name, st);
    hipLaunchKernelGGL((ntt_fp_kernel<K3, MODE, COLUMNS>), grid, dim3(threads), lds, st, a, g, (int)tasks);
    return hipGetLastError();
}

// Rows by four waves or by one: up to about eight waves a SIMD of the former (inverse rows 64: 5.8 -> 4.0 us, 1088: 9.3 -> 7.4, 2176:
// 12.7 -> 10.2, 4352: 18.1 -> 18.4, 26112: 76 -> 93; rows of a rescale 192: 6.5 -> 4.9, 2048: 12.6 -> 11.6, 2816: 13.4 -> 14.0, 16384:
// 65 -> 89: four exchanges a row instead of two).  Inner products: while all workgroups are resident at once, 512 of eight waves (up to
// two digits) or 256 of twelve or sixteen (two digits 24: 8.9 -> 8.0 us, 384: 13.8 -> 12.7, 768: 16.3 -> 18.0; three digits 128: 12.1 -> 9.4,
// 256: 13.2 -> 10.7, 736: 21 -> 26; four digits 256: 14.9 -> 11.4, 320: 19.3 -> 20.1).  Of these a workgroup for each polynomial while both fit
// the chip's 256 compute units (WIDE_SPLIT): one rotation at N = 2^13, 8 limbs, 26.3 -> 25.6 us; whole rotations with 32, 64, 96 and 128 tasks
// of one digit 22.3, 22.5, 22.9, 23.1 -> 21.3, 21.4, 21.9, 22.1, of three digits 23.9 .. 25.6 -> 23.3 .. 24.7; behind the line, 144 to 192
// tasks, as without.
// Forward transforms with their columns, us, 8-byte rows by one wave / 16-byte ones / these: 1280 rows at N = 2^14 13.5 / 14.2 / 12.5, 2048
// 15.5 / 16.3 / 16.0; of 4096, the one place where 16-byte rows lose (two exchanges of lanes a row, nothing to hide them behind), 23.0 / 24.1,
// of 6144 and more even.
#define WIDE_ROWS 2048
static u64 wide_inner_tasks(int n_digits) { return n_digits > WIDE_DIGITS ? 0 : n_digits <= 2 ? 512 : 256; }
template <int K3, int MODE>
static hipError_t launch_wide_k3(const ConvertArgs& a, const InnerArgs& g, u64 tasks, hipStream_t st) {
    static char name[40] = "";
    if (!name[0]) snprintf(name, sizeof name, "ntt_fp_wide_kernel<%d, %d>", K3, MODE);
    InnerArgs ga = g;
    ga.split = fp_inner(MODE) && 2 * tasks <= WIDE_SPLIT;
    const unsigned digits = (unsigned)a.n_digits, rows = !fp_inner(MODE) ? 1 : ga.split ? std::min(digits + 1, (unsigned)WIDE_DIGITS) : std::max(digits, 2u);
    tasks <<= ga.split;
    ProfScope prof__(name, st);
    hipLaunchKernelGGL((ntt_fp_wide_kernel<K3, MODE>), dim3((unsigned)((tasks + 7) / 8 * 8)), dim3(rows * WIDE_NT), rows * WIDE_LDS * 8, st, a, ga,
                       (int)tasks);
    return hipGetLastError();
}

template <int MODE>
static hipError_t launch_rows(const ConvertArgs& a, const InnerArgs& g, u64 limbs, hipStream_t st) {
    const u64 tasks = (limbs * a.n_entries) << (a.log_n - 10);
    if (tasks > 0x7fffff00u) return hipErrorInvalidValue;
    if (tasks <= (fp_inner(MODE) ? wide_inner_tasks(a.n_digits) : WIDE_ROWS)) {
        switch (a.log_n) {
            case 12: return launch_wide_k3<2, MODE>(a, g, tasks, st);
            case 13: return launch_wide_k3<3, MODE>(a, g, tasks, st);
            case 14: return launch_wide_k3<4, MODE>(a, g, tasks, st);
            default: return launch_wide_k3<5, MODE>(a, g, tasks, st);
        }
    }
    constexpr unsigned threads = fp_threads(MODE, false);
    const u64 per_block = threads == 128 ? 1 : threads / 64;     // a pair of waves shares a task of the inner products
    const dim3 grid((unsigned)(((tasks + per_block - 1) / per_block + 7) / 8 * 8));
    switch (a.log_n) {
        case 12: return launch_one<2, MODE, false>(grid, threads, 0, a, g, tasks, st);
        case 13: return launch_one<3, MODE, false>(grid, threads, 0, a, g, tasks, st);
        case 14: return launch_one<4, MODE, false>(grid, threads, 0, a, g, tasks, st);
        default: return launch_one<5, MODE, false>(grid, threads, 0, a, g, tasks, st);
    }
}

static hipError_t launch_step_rows_once(int mode, dim3 grid, const ConvertArgs& a, const InnerArgs& g, const StepArgs& s, int tasks, hipStream_t st);
template <int MODE>
static hipError_t launch_step_rows(const ConvertArgs& a, const InnerArgs& g, const StepArgs& s, u64 limbs, hipStream_t st) {
    const u64 tasks = (limbs * a.n_entries) << (a.log_n - 10);
    if (tasks > 0x7fffff00u) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((tasks + 7) / 8 * 8));
    ProfScope prof__("inner_product_steps_rows_kernel", st);
    if (s.step_B == 1 && (((u64)a.ext_limbs * a.n_digits * 2 * a.n_entries) << (a.log_n + 3)) > STREAMED_KEY_BYTES)
        return launch_step_rows_once(MODE, grid, a, g, s, (int)tasks, st);
#define STEPS_CASE(K3)                                                                                                            \
    case 10 + K3:                                                                                                                 \
        hipLaunchKernelGGL((inner_product_steps_rows_kernel<K3, MODE, false>), grid, dim3(128), 0, st, a, g, s, (int)tasks);      \
        break;
    switch (a.log_n) {
        STEPS_CASE(2) STEPS_CASE(3) STEPS_CASE(4) STEPS_CASE(5)
        default: return hipErrorInvalidValue;
    }
#undef STEPS_CASE
    return hipGetLastError();
}

template <int K3, int MODE>
static hipError_t launch_columns_k3(const ConvertArgs& a_in, hipStream_t st) {
    ConvertArgs a = a_in;
    constexpr int NR = Col<K3>::NR, TILES = 1024 / Col<K3>::WIDTH;
    constexpr int PER_SRC = NR * 64 * 8, MAX_CHUNK = 20 * 8192 / PER_SRC;
    constexpr int MOST_SOURCES = HISA_MAX_PRIMES / 2 + 1;        // as many special primes as primes, and the last prime
    int most = 1;
    for (int d = 0; d < a.n_digits; d++) most = a.dg[d].a > most ? a.dg[d].a : most;
    a.chunk = most < MAX_CHUNK ? most : MAX_CHUNK;
    const size_t lds = (size_t)a.chunk * PER_SRC;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)ntt_fp_kernel<K3, MODE, true>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           MAX_CHUNK * PER_SRC);
        if constexpr (MAX_CHUNK < MOST_SOURCES)
            if (e == hipSuccess)
                e = hipFuncSetAttribute((const void*)ntt_fp_chunks_kernel<K3, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize, MAX_CHUNK * PER_SRC);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    // Sixteen waves where only one workgroup fits a compute unit's LDS (more than 80 KB of sources: 10 of them from N = 2^14
    // on, 20 at 2^13), else eight.  rotLeft in us, eight -> sixteen waves, batches of 64, 16 and 1.  Above the line: 11 sources at
    // N = 2^15 1893 -> 1835, 515 -> 490, 70 -> 74; 16 sources 1473 -> 1438, 394 -> 381, 69 -> 81; 16 at N = 2^14 715 -> 737,
    // 198 -> 191, 61 -> 74; 21 at N = 2^13 562 -> 522, 163 -> 148, 50 -> 53: single ciphertexts would be served better by eight.
    // Below it: 8 sources at N = 2^15 611 -> 649, 171 -> 178, 51 -> 50; 7 sources 1768 -> 1817, 479 -> 496, 72 -> 70.
    const unsigned threads = lds > 81920 ? 1024 : 512;
    // Few entries: several workgroups share a tile's targets (each forms the conversion inputs for itself), so that the
    // launch reaches about two workgroups per compute unit before a workgroup takes a second round of targets.
    const int waves = (int)(threads / 64);
    int rounds = 1;
    for (int d = 0; d < a.n_digits; d++) {
        const int r = (a.ext_limbs - a.dg[d].own_n + waves - 1) / waves;
        rounds = r > rounds ? r : rounds;
    }
    a.n_splits = 1;
    while (a.n_splits < rounds && (u64)a.n_entries * a.n_digits * TILES * (a.n_splits + 1) <= 512) a.n_splits++;
    // a grid has at most 65535 rows of entries: a larger batch takes several launches
    for (unsigned e0 = 0; e0 < a_in.n_entries; e0 += 65535) {
        a.n_entries = a_in.n_entries - e0 < 65535 ? a_in.n_entries - e0 : 65535;
        a.mid = a_in.mid + (u64)e0 * a.n_src * ((u64)1 << a.log_n);
        a.out = a_in.out + (u64)e0 * a.out_bs;
        const dim3 grid((unsigned)(TILES * a.n_digits * a.n_splits), a.n_entries);
        hipError_t e = hipErrorInvalidValue;
        if (most <= MAX_CHUNK) {
            e = launch_one<K3, MODE, true>(grid, threads, lds, a, InnerArgs{}, 0, st);
        } else if constexpr (MAX_CHUNK < MOST_SOURCES) {
            static char name[40] = "";
            if (!name[0]) snprintf(name, sizeof name, "ntt_fp_chunks_kernel<%d, %d>", K3, MODE);
            ProfScope prof__(name, st);
            hipLaunchKernelGGL((ntt_fp_chunks_kernel<K3, MODE>), grid, dim3(threads), lds, st, a);
            e = hipGetLastError();
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int MODE>
static hipError_t launch_columns(const ConvertArgs& a, hipStream_t st) {
    switch (a.log_n) {
        case 12: return launch_columns_k3<2, MODE>(a, st);
        case 13: return launch_columns_k3<3, MODE>(a, st);
        case 14: return launch_columns_k3<4, MODE>(a, st);
        default: return launch_columns_k3<5, MODE>(a, st);
    }
}

hipError_t launch_inverse_rows_fp(const ConvertArgs& a, hipStream_t st) {
    DRY_RUN_RETURN();
    if (a.n_entries == 0) return hipSuccess;
    u64 targets = 0;
    if (!convert_args_ok(a, &targets) || !a.in) return hipErrorInvalidValue;
    return launch_rows<FP_INV_TO_Y>(a, InnerArgs{}, (u64)a.n_src, st);
}

hipError_t launch_columns_fp(int mode, const ConvertArgs& a, hipStream_t st) {
    DRY_RUN_RETURN();
    if (a.n_entries == 0) return hipSuccess;
    u64 targets = 0;
    if (!convert_args_ok(a, &targets)) return hipErrorInvalidValue;
    switch (mode) {
        case FP_FWD_CONV: return launch_columns<FP_FWD_CONV>(a, st);
        case FP_FWD_CONV_FINAL: return launch_columns<FP_FWD_CONV_FINAL>(a, st);
        case FP_FWD_CONV_SUB: return launch_columns<FP_FWD_CONV_SUB>(a, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_forward_rows_fp(int mode, const ConvertArgs& a, hipStream_t st) {
    DRY_RUN_RETURN();
    if (a.n_entries == 0) return hipSuccess;
    u64 targets = 0;
    if (!convert_args_ok(a, &targets)) return hipErrorInvalidValue;
    if (mode != FP_FWD_CONV && (!a.acc || a.n_digits != 1)) return hipErrorInvalidValue;
    if (mode == FP_FWD_CONV_FINAL) {
        if (!a.pinv_tab || (a.add && a.add_div <= 0)) return hipErrorInvalidValue;
    }
    switch (mode) {
        case FP_FWD_CONV: return launch_rows<FP_FWD_CONV>(a, InnerArgs{}, targets, st);
        case FP_FWD_CONV_FINAL: return launch_rows<FP_FWD_CONV_FINAL>(a, InnerArgs{}, targets, st);
        case FP_FWD_SUB: return launch_rows<FP_FWD_SUB>(a, InnerArgs{}, targets, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_inner_rows_fp(int mode, const ConvertArgs& a, const InnerArgs& g, const StepArgs* steps, hipStream_t st) {
    DRY_RUN_RETURN();
    if (a.n_entries == 0) return hipSuccess;
    u64 targets = 0;
    if (!convert_args_ok(a, &targets)) return hipErrorInvalidValue;
    const u64 n = (u64)1 << a.log_n;
    if (steps) {        // every entry belongs to a rotation with its key and Galois element
        if (steps->step_B < 1 || a.n_entries % steps->step_B || a.n_entries / steps->step_B > FP_MAX_STEPS) return hipErrorInvalidValue;
        for (unsigned s = 0; s < a.n_entries / steps->step_B; s++)
            if (!steps->steps.key[s] || steps->steps.galois[s] == 0) return hipErrorInvalidValue;
    }
    if ((!steps && !g.key) || !g.own || !g.c1 || g.n_acc < 1 || g.n_acc >= a.ext_limbs || g.n_acc > a.l) return hipErrorInvalidValue;
    if (g.x_begin < 0 || g.x_begin >= g.x_end || g.x_end > a.ext_limbs) return hipErrorInvalidValue;
    if (g.own_bs < (u64)a.l * n || g.add_polys < 0 || g.add_polys > 2 || (g.add_polys && !g.add)) return hipErrorInvalidValue;
    if (g.add_polys && (g.add_bs < (u64)g.add_polys * a.l * n || (g.add_polys > 1 && g.add_ps < (u64)a.l * n))) return hipErrorInvalidValue;
    const u64 limbs = (u64)(g.x_end - g.x_begin);
    if (mode == FP_INV_D_TO_Y) {
        if ((g.x_begin < g.n_acc && !g.acc) || (g.x_end > g.n_acc && !g.down)) return hipErrorInvalidValue;
        return steps ? launch_step_rows<FP_INV_D_TO_Y>(a, g, *steps, limbs, st) : launch_rows<FP_INV_D_TO_Y>(a, g, limbs, st);
    }
    if (mode != FP_FWD_CONV_SUB || g.x_end > g.n_acc || !g.out) return hipErrorInvalidValue;
    return steps ? launch_step_rows<FP_FWD_CONV_SUB>(a, g, *steps, limbs, st) : launch_rows<FP_FWD_CONV_SUB>(a, g, limbs, st);
}

// ---- whole polynomials ----
template <int MODE>
static hipError_t launch_split(int log_n, FpArgs a, const FpTask& tk, bool columns, hipStream_t st) {
    const u64 polys = (u64)tk.period * a.n_entries;
    const int tiles = log_n == 15 ? 32 : 16;
    a.n_tasks = (int)(columns ? polys * tiles : polys << (log_n - 10));
    const bool wide = !columns && a.n_tasks <= WIDE_ROWS;
    const dim3 grid((unsigned)((((u64)a.n_tasks + (wide ? 0 : 3)) / (wide ? 1 : 4) + 7) / 8 * 8));
    static char names[4][3][40];
    char* name = names[log_n - 12][wide ? 2 : columns];
    if (!name[0] && wide) snprintf(name, 40, "ntt_fp_split_wide_kernel<%d, %d>", log_n - 10, MODE);
    else if (!name[0]) snprintf(name, 40, "ntt_fp_split_kernel<%d, %d, %s>", log_n - 10, MODE, columns ? "true" : "false");
    ProfScope prof__(name, st);
#define SPLIT_CASE(K3)                                                                                             \
    case 10 + K3:                                                                                                  \
        if (columns) hipLaunchKernelGGL((ntt_fp_split_kernel<K3, MODE, true>), grid, dim3(ROWS_NT), 0, st, a, tk); \
        else if (wide) hipLaunchKernelGGL((ntt_fp_split_wide_kernel<K3, MODE>), grid, dim3(WIDE_NT), 0, st, a, tk); \
        else hipLaunchKernelGGL((ntt_fp_split_kernel<K3, MODE, false>), grid, dim3(ROWS_NT), 0, st, a, tk);        \
        break;
    switch (log_n) {
        SPLIT_CASE(2) SPLIT_CASE(3) SPLIT_CASE(4) SPLIT_CASE(5)
        default: return hipErrorInvalidValue;
    }
#undef SPLIT_CASE
    return hipGetLastError();
}

hipError_t launch_ntt_fp_split(int mode, int log_n, const FpArgs& a_in, const FpTask& tk, u64 n_batch, hipStream_t st) {
    FpArgs a = a_in;
    if (log_n < 12 || log_n > 15 || !a.sfwd || !a.sinv || !a.out || n_batch == 0 || ((u64)tk.period * n_batch << (log_n - 5)) > 0x7fffff00u)
        return hipErrorInvalidValue;
    a.n_entries = (int)n_batch;
    a.table_stride = split_table_words(log_n);
    hipError_t e;
    if (mode == FP_INV_PLAIN) {
        if (!a.in) return hipErrorInvalidValue;
        e = launch_split<FP_INV_PLAIN>(log_n, a, tk, false, st);
        return e == hipSuccess ? launch_split<FP_INV_PLAIN>(log_n, a, tk, true, st) : e;
    }
    if (mode != FP_FWD_PLAIN || (!a.in && !a.coeffs)) return hipErrorInvalidValue;
    e = launch_split<FP_FWD_PLAIN>(log_n, a, tk, true, st);
    return e == hipSuccess ? launch_split<FP_FWD_PLAIN>(log_n, a, tk, false, st) : e;
}

template <int K3>
static hipError_t launch_encrypt_k3(const EncryptArgs& a, hipStream_t st) {
    const u64 cols = (u64)a.n_entries * a.limbs * 2 * (1024 / Col<K3>::WIDTH), rows = ((u64)a.n_entries * a.limbs) << K3;
    {
        ProfScope prof__("encrypt_columns_kernel", st);
        hipLaunchKernelGGL(encrypt_columns_kernel<K3>, dim3((unsigned)(((cols + 3) / 4 + 7) / 8 * 8)), dim3(ROWS_NT), 0, st, a);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (rows <= WIDE_ROWS / 2) {
        ProfScope prof__("encrypt_rows_wide_kernel", st);
        hipLaunchKernelGGL(encrypt_rows_wide_kernel<K3>, dim3((unsigned)((rows + 7) / 8 * 8)), dim3(2 * WIDE_NT), 0, st, a);
        return hipGetLastError();
    }
    ProfScope prof__("encrypt_rows_kernel", st);
    hipLaunchKernelGGL(encrypt_rows_kernel<K3>, dim3((unsigned)(((rows + 3) / 4 + 7) / 8 * 8)), dim3(ROWS_NT), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_encrypt_fp(int log_n, const EncryptArgs& a_in, hipStream_t st) {
    DRY_RUN_RETURN();
    EncryptArgs a = a_in;
    if (!a.fprimes || !a.primes || !a.sfwd || !a.secret || !a.ct || a.limbs < 1 || a.n_entries < 1 || a.n_entries > ENCRYPT_MAX ||
        (a.noise_on && (!a.cdt || a.cdt_n < 1)))
        return hipErrorInvalidValue;
    for (int b = 0; b < a.n_entries; b++)
        if (!a.pt[b]) return hipErrorInvalidValue;
    a.table_stride = split_table_words(log_n);
    switch (log_n) {
        case 12: return launch_encrypt_k3<2>(a, st);
        case 13: return launch_encrypt_k3<3>(a, st);
        case 14: return launch_encrypt_k3<4>(a, st);
        case 15: return launch_encrypt_k3<5>(a, st);
        default: return hipErrorInvalidValue;
    }
}

// Keys that pass the caches by.  The last launches of this file, so that their kernels lie behind all others: where a kernel lies in
// the code object moves its time by up to 1 % (37 products relinearised at N = 2^14, 11 limbs, the same instructions behind 0 .. 64 KB of
// padding, 407 .. 410 us; 38 rotations at N = 2^13, 3 limbs, 66.3 .. 67.6), and the kernels of every other call need not lie farther apart.
static hipError_t launch_step_rows_once(int mode, dim3 grid, const ConvertArgs& a, const InnerArgs& g, const StepArgs& s, int tasks, hipStream_t st) {
#define ONCE_CASE(K3, MODE)                                                                                                    \
    if (a.log_n == 10 + K3 && mode == MODE) {                                                                                  \
        hipLaunchKernelGGL((inner_product_steps_rows_kernel<K3, MODE, true>), grid, dim3(128), 0, st, a, g, s, tasks);         \
        return hipGetLastError();                                                                                              \
    }
    ONCE_CASE(2, FP_INV_D_TO_Y) ONCE_CASE(3, FP_INV_D_TO_Y) ONCE_CASE(4, FP_INV_D_TO_Y) ONCE_CASE(5, FP_INV_D_TO_Y)
    ONCE_CASE(2, FP_FWD_CONV_SUB) ONCE_CASE(3, FP_FWD_CONV_SUB) ONCE_CASE(4, FP_FWD_CONV_SUB) ONCE_CASE(5, FP_FWD_CONV_SUB)
#undef ONCE_CASE
    return hipErrorInvalidValue;
}
