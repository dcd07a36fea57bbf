// Sampling and limb-wise kernels: the counter-based generator with its
// uniform / ternary / discrete-Gaussian samplers, add / sub / mulPlain /
// mulScalar / mulNoRelin, the combine steps of encryption, decryption and key
// generation, and the NTT-form automorphism gather.  All of them stream
// [..][limb][N] arrays once: they are bound by HBM bandwidth.
#include "hisa_internal.hpp"
#include "modarith.hpp"
#include "fparith.hpp"
#include "sampling.hpp"

#define NT 256

// Two coefficients a thread, 16 bytes an access (polynomials start at multiples of 8 KB of a pool block), and where a kernel
// treats several polynomials alike, all of them: 24 products of two polynomials at N = 2^14, 8 limbs were 24576 workgroups of 2 KB
// each way, 23 us, and are 18 now; the sums 25 us, 22 now.  Beyond the last-level cache that is not the better form everywhere (launch_addsub,
// launch_mul_no_relin).
typedef u64 u64x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u64x2 ld2(const u64* p) { return *(const u64x2*)p; }
__device__ __forceinline__ void st2(u64* p, u64x2 v) { *(u64x2*)p = v; }
// what a launch reads and writes, in polynomials of one limb, does not fit the last-level cache
static bool beyond_cache(u64 limb_polys, int log_n) { return limb_polys << (log_n + 3) > (u64)256 << 20; }
#define PAIR_BLOCKS(log_n) ((1u << (log_n)) / (2 * NT))
__device__ __forceinline__ u64 pair_at() { return 2 * ((u64)blockIdx.x * NT + threadIdx.x); }

__global__ __launch_bounds__(NT) void sample_uniform_kernel(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr,
                                                            PolyMap map, u64 batch_stride, u64 ctr_step, u64* out,
                                                            int log_n) {
    const u64 n = (u64)1 << log_n;
    const int p = blockIdx.y, entry = p % map.period, b = p / map.period;
    const int prime = map.prime_of[entry];
    if (prime < 0) return;
    const PrimeConst pc = primes[prime];
    const u64 key = stream_key(seed, kind, ctr + (u64)b * ctr_step);
    u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    u64 w = rnd_at(key, (u64)prime * n + j);
    out[(u64)b * batch_stride + (u64)entry * n + j] = barrett128(0, w, pc.q, pc.r1, pc.r0);
}

hipError_t launch_sample_uniform(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr, const PolyMap& map, int n_polys,
                                 u64 batch_stride, u64 ctr_step, u64* out, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    dim3 grid((1u << log_n) / NT, n_polys);
    ProfScope prof__("sample_uniform_kernel", st);
    hipLaunchKernelGGL(sample_uniform_kernel, grid, dim3(NT), 0, st, primes, seed, kind, ctr, map, batch_stride, ctr_step,
                       out, log_n);
    return hipGetLastError();
}

// One small signed polynomial per batch entry (ternary secret, or Gaussian
// error, or zero), reduced into every mapped limb.  raw (may be null) receives
// the signed coefficients of batch entry 0.  cdt[k] = floor(2^63 * P(|X| <= k)), k < cdt_n, of the context's
// error distribution: the magnitude is the number of entries the word's upper 63 bits reach, the sign its low bit.
__global__ __launch_bounds__(NT) void sample_small_kernel(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr,
                                                          int noise_on, int ternary, const u64* cdt, int cdt_n, PolyMap map,
                                                          u64 batch_stride, u64 ctr_step, u64* out, i64* raw, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int b = blockIdx.y;
    const u64 key = stream_key(seed, kind, ctr + (u64)b * ctr_step);
    const u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    const u64 w = rnd_at(key, j);
    i64 v;
    if (ternary) {
        u64 t = w % 3;
        v = t == 0 ? 0 : (t == 1 ? 1 : -1);
    } else if (noise_on) {
        v = gaussian_from_word(w, cdt, cdt_n);
    } else {
        v = 0;
    }
    if (raw && b == 0) raw[j] = v;
    for (int e = 0; e < map.period; e++) {
        int prime = map.prime_of[e];
        if (prime < 0) continue;
        u64 q = primes[prime].q;
        out[(u64)b * batch_stride + (u64)e * n + j] = v >= 0 ? (u64)v : q - (u64)(-v);
    }
}

hipError_t launch_sample_small(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr, int noise_on, int ternary,
                               const u64* cdt, int cdt_n, const PolyMap& map, int n_polys, u64 batch_stride, u64 ctr_step,
                               u64* out, i64* raw, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (!ternary && noise_on && (!cdt || cdt_n <= 0)) return hipErrorInvalidValue;
    dim3 grid((1u << log_n) / NT, n_polys);  // n_polys = batch entries here
    ProfScope prof__("sample_small_kernel", st);
    hipLaunchKernelGGL(sample_small_kernel, grid, dim3(NT), 0, st, primes, seed, kind, ctr, noise_on, ternary, cdt, cdt_n,
                       map, batch_stride, ctr_step, out, raw, log_n);
    return hipGetLastError();
}

// ---- add / sub --------------------------------------------------------------
// out[b][p][i] = a[b][p][i] (+|-) b[b][p][i] for p < polys_b, copy of a for the rest.  A workgroup: `polys` of the polynomials
__global__ __launch_bounds__(NT) void addsub_kernel(const PrimeConst* primes, const u64* a, const u64* b, u64* out, int op,
                                                    int limbs, int polys, int polys_a, int polys_b, u64 a_bs, u64 b_bs, u64 o_bs,
                                                    int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y % limbs, first = blockIdx.y / limbs * polys, end = first + polys;
    const u64 bi = blockIdx.z;
    const u64 q = primes[limb].q;
    const u64 j = (u64)limb * n + pair_at();
    // two polynomials' loads ahead of the first store: a small call waits once
    for (int poly = first; poly < end; poly += 2) {
        u64x2 x[2], y[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const u64 off = (u64)(poly + k) * limbs * n + j;
            if (poly + k < end) x[k] = ld2(a + bi * a_bs + off);
            if (poly + k < end && poly + k < polys_b) y[k] = ld2(b + bi * b_bs + off);
        }
#pragma unroll
        for (int k = 0; k < 2; k++) {
            if (poly + k >= end) break;
            if (poly + k < polys_b)
                x[k] = op == OP_ADD ? u64x2{addmod(x[k].x, y[k].x, q), addmod(x[k].y, y[k].y, q)} : u64x2{submod(x[k].x, y[k].x, q), submod(x[k].y, y[k].y, q)};
            st2(out + bi * o_bs + (u64)(poly + k) * limbs * n + j, x[k]);
        }
    }
}

hipError_t launch_addsub(const PrimeConst* primes, const u64* a, const u64* b, u64* out, int op, int limbs, int polys_a,
                         int polys_b, u64 n_batch, u64 a_bs, u64 b_bs, u64 o_bs, int log_n, hipStream_t st) {
    if (t_analysis) TALLY(add, HISA_OP_ADD, n_batch, limbs);
    DRY_RUN_RETURN();
    // All polynomials of an entry in a workgroup, or beyond the cache one: us, 64 sums at N = 2^15, 16 limbs 291 -> 285, and 308 -> 303 where
    // a rescale follows; 60 at 9 limbs 163 -> 159 so; 96 at N = 2^14, 12 limbs 156 -> 153; 64 at N = 2^12, 16 limbs (200 MB) even.
    const int polys = beyond_cache(3 * (u64)polys_a * limbs * n_batch, log_n) ? 1 : polys_a;
    dim3 grid(PAIR_BLOCKS(log_n), limbs * (polys_a / polys), (unsigned)n_batch);
    ProfScope prof__("addsub_kernel", st);
    hipLaunchKernelGGL(addsub_kernel, grid, dim3(NT), 0, st, primes, a, b, out, op, limbs, polys, polys_a, polys_b, a_bs, b_bs,
                       o_bs, log_n);
    return hipGetLastError();
}

struct LimbConsts {
    u64 v[HISA_MAX_PRIMES];
    u64 v_sh[HISA_MAX_PRIMES];
};

// first polynomial +- per-limb constant (a constant polynomial is that constant at every evaluation point)
__global__ __launch_bounds__(NT) void add_const_kernel(const PrimeConst* primes, const u64* a, u64* out, LimbConsts c,
                                                       int op, int limbs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y % limbs, poly = blockIdx.y / limbs;
    const u64 q = primes[limb].q;
    const u64 off = ((u64)poly * limbs + limb) * n + (u64)blockIdx.x * NT + threadIdx.x;
    u64 x = a[off];
    if (poly == 0) x = op == OP_ADD ? addmod(x, c.v[limb], q) : submod(x, c.v[limb], q);
    out[off] = x;
}

hipError_t launch_add_const(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int op, int limbs,
                            int polys, int log_n, hipStream_t st) {
    if (t_analysis) TALLY(add, HISA_OP_ADD, (polys + 1) / 2, limbs);
    DRY_RUN_RETURN();
    LimbConsts c = {};
    for (int i = 0; i < limbs; i++) c.v[i] = consts[i];
    dim3 grid((1u << log_n) / NT, limbs * polys);
    ProfScope prof__("add_const_kernel", st);
    hipLaunchKernelGGL(add_const_kernel, grid, dim3(NT), 0, st, primes, a, out, c, op, limbs, log_n);
    return hipGetLastError();
}

// ---- multiply ---------------------------------------------------------------
// batch entry b is multiplied by plaintext b % pt_period (plaintexts [limbs][N], one after the other)
__global__ __launch_bounds__(NT) void mul_plain_kernel(const PrimeConst* primes, const u64* a, const u64* pt, u64* out,
                                                       int limbs, int polys, u64 a_bs, u64 o_bs, unsigned pt_period, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 bi = blockIdx.z;
    const PrimeConst pc = primes[limb];
    const u64 j = (u64)limb * n + pair_at();
    const u64x2 w = ld2(pt + (bi % pt_period) * (u64)limbs * n + j);
    for (int poly = 0; poly < polys; poly += 2) {
        u64x2 x[2];
#pragma unroll
        for (int k = 0; k < 2; k++)
            if (poly + k < polys) x[k] = ld2(a + bi * a_bs + (u64)(poly + k) * limbs * n + j);
#pragma unroll
        for (int k = 0; k < 2; k++)
            if (poly + k < polys)
                st2(out + bi * o_bs + (u64)(poly + k) * limbs * n + j,
                    u64x2{mulmod_barrett(x[k].x, w.x, pc.q, pc.r1, pc.r0), mulmod_barrett(x[k].y, w.y, pc.q, pc.r1, pc.r0)});
    }
}

hipError_t launch_mul_plain(const PrimeConst* primes, const u64* a, const u64* pt, u64* out, int limbs, int polys,
                            u64 n_batch, u64 a_bs, u64 o_bs, int log_n, hipStream_t st, unsigned pt_period) {
    if (t_analysis) TALLY(mul_plain, HISA_OP_MUL_PLAIN, n_batch, limbs);
    DRY_RUN_RETURN();
    if (pt_period == 0 || n_batch == 0 || n_batch > 65535) return hipErrorInvalidValue;
    dim3 grid(PAIR_BLOCKS(log_n), limbs, (unsigned)n_batch);
    ProfScope prof__("mul_plain_kernel", st);
    hipLaunchKernelGGL(mul_plain_kernel, grid, dim3(NT), 0, st, primes, a, pt, out, limbs, polys, a_bs, o_bs, pt_period, log_n);
    return hipGetLastError();
}

__global__ __launch_bounds__(NT) void mul_const_kernel(const PrimeConst* primes, const u64* a, u64* out, LimbConsts c,
                                                       int limbs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y % limbs;
    const u64 q = primes[limb].q;
    const u64 off = (u64)blockIdx.y * n + pair_at();
    const u64x2 x = ld2(a + off);
    st2(out + off, u64x2{shoup_mul(x.x, c.v[limb], c.v_sh[limb], q), shoup_mul(x.y, c.v[limb], c.v_sh[limb], q)});
}

hipError_t launch_mul_const(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int limbs, int polys,
                            int log_n, hipStream_t st) {
    if (t_analysis) TALLY(mul_scalar, HISA_OP_MUL_SCALAR, (polys + 1) / 2, limbs);
    DRY_RUN_RETURN();
    // consts: [limbs] values followed by [limbs] Shoup companions
    LimbConsts c = {};
    for (int i = 0; i < limbs; i++) { c.v[i] = consts[i]; c.v_sh[i] = consts[limbs + i]; }
    dim3 grid(PAIR_BLOCKS(log_n), limbs * polys);
    ProfScope prof__("mul_const_kernel", st);
    hipLaunchKernelGGL(mul_const_kernel, grid, dim3(NT), 0, st, primes, a, out, c, limbs, log_n);
    return hipGetLastError();
}

// (a0, a1) x (b0, b1) -> (a0 b0, a0 b1 + a1 b0, a1 b1)
__global__ __launch_bounds__(NT) void mul_no_relin_kernel(const PrimeConst* primes, const u64* a, const u64* b, u64* out,
                                                          int limbs, u64 a_bs, u64 b_bs, u64 o_bs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 bi = blockIdx.z;
    const PrimeConst pc = primes[limb];
    const u64 j = pair_at();
    const u64 o0 = (u64)limb * n + j, o1 = ((u64)limbs + limb) * n + j, o2 = ((u64)2 * limbs + limb) * n + j;
    const u64x2 a0 = ld2(a + bi * a_bs + o0), a1 = ld2(a + bi * a_bs + o1);
    const u64x2 b0 = ld2(b + bi * b_bs + o0), b1 = ld2(b + bi * b_bs + o1);
    auto product = [&](u64 x, u64 y) { return mulmod_barrett(x, y, pc.q, pc.r1, pc.r0); };
    auto cross = [&](u64 x0, u64 y1, u64 x1, u64 y0) {
        Acc128 acc = {0, 0};
        acc_mad(acc, x0, y1);
        acc_mad(acc, x1, y0);
        return acc_reduce(acc, pc.q, pc.r1, pc.r0);
    };
    st2(out + bi * o_bs + o0, u64x2{product(a0.x, b0.x), product(a0.y, b0.y)});
    st2(out + bi * o_bs + o1, u64x2{cross(a0.x, b1.x, a1.x, b0.x), cross(a0.y, b1.y, a1.y, b0.y)});
    st2(out + bi * o_bs + o2, u64x2{product(a1.x, b1.x), product(a1.y, b1.y)});
}

// The same beyond the cache: a coefficient a thread, workgroups of 8 KB, and the two polynomials that relinearisation reads last leave
// past the caches.
#define MUL_STREAM_NT 1024
__global__ __launch_bounds__(MUL_STREAM_NT) void mul_no_relin_stream_kernel(const PrimeConst* primes, const u64* a, const u64* b, u64* out,
                                                                            int limbs, u64 a_bs, u64 b_bs, u64 o_bs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 bi = blockIdx.z;
    const PrimeConst pc = primes[limb];
    const u64 j = (u64)blockIdx.x * MUL_STREAM_NT + threadIdx.x;
    const u64 o0 = (u64)limb * n + j, o1 = ((u64)limbs + limb) * n + j, o2 = ((u64)2 * limbs + limb) * n + j;
    const u64 a0 = a[bi * a_bs + o0], a1 = a[bi * a_bs + o1];
    const u64 b0 = b[bi * b_bs + o0], b1 = b[bi * b_bs + o1];
    __builtin_nontemporal_store(mulmod_barrett(a0, b0, pc.q, pc.r1, pc.r0), out + bi * o_bs + o0);
    Acc128 acc = {0, 0};
    acc_mad(acc, a0, b1);
    acc_mad(acc, a1, b0);
    __builtin_nontemporal_store(acc_reduce(acc, pc.q, pc.r1, pc.r0), out + bi * o_bs + o1);
    out[bi * o_bs + o2] = mulmod_barrett(a1, b1, pc.q, pc.r1, pc.r0);
}

hipError_t launch_mul_no_relin(const PrimeConst* primes, const u64* a, const u64* b, u64* out, int limbs, u64 n_batch,
                               u64 a_bs, u64 b_bs, u64 o_bs, int log_n, hipStream_t st) {
    if (t_analysis) TALLY(mul, HISA_OP_MUL, n_batch, limbs);
    DRY_RUN_RETURN();
    // Bound by memory: seven streams.  Two coefficients a thread in workgroups of 4 KB -> one in 8 KB past the caches, us: 32 products at
    // N = 2^14, 12 limbs 63 -> 53, 64 123 -> 119, 96 180 -> 179 (one coefficient in 2 KB: 60, 119, 177); at N = 2^15, 16 limbs 16 86 -> 80, 64
    // 340 -> 326 (379); 24 at N = 2^14, 11 limbs (231 MB) 37.9 either way.  37 there with relinearisation and rescale 432 -> 423.  A batch's
    // squares read two polynomials fewer and stay with pairs: 64 at N = 2^15, 16 limbs 237 against 261.
    if (a != b && beyond_cache((u64)7 * limbs * n_batch, log_n)) {
        dim3 grid((1u << log_n) / MUL_STREAM_NT, limbs, (unsigned)n_batch);
        ProfScope prof__("mul_no_relin_stream_kernel", st);
        hipLaunchKernelGGL(mul_no_relin_stream_kernel, grid, dim3(MUL_STREAM_NT), 0, st, primes, a, b, out, limbs, a_bs, b_bs, o_bs, log_n);
        return hipGetLastError();
    }
    dim3 grid(PAIR_BLOCKS(log_n), limbs, (unsigned)n_batch);
    ProfScope prof__("mul_no_relin_kernel", st);
    hipLaunchKernelGGL(mul_no_relin_kernel, grid, dim3(NT), 0, st, primes, a, b, out, limbs, a_bs, b_bs, o_bs, log_n);
    return hipGetLastError();
}

// x^2 + c x before relinearisation, (a0 (a0 + c), a1 (2 a0 + c), a1^2): what an activation starts from, in one pass over x.
// Product, scaled copy and sum as launches of their own moved 15 polynomials where this moves five; bound by memory.
// All activations of a network, us: LeNet-medium 286 -> 94, SqueezeNet-style 442 -> 140 (and 16 copies of concatenated inputs).
__global__ __launch_bounds__(NT) void square_linear_kernel(const PrimeConst* primes, const u64* a, u64* out, LimbConsts c, int limbs,
                                                           u64 a_bs, u64 o_bs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 bi = blockIdx.z;
    const PrimeConst pc = primes[limb];
    const u64 j = pair_at();
    const u64 o0 = (u64)limb * n + j, o1 = ((u64)limbs + limb) * n + j, o2 = ((u64)2 * limbs + limb) * n + j;
    const u64x2 a0 = ld2(a + bi * a_bs + o0), a1 = ld2(a + bi * a_bs + o1);
    const u64x2 s = {addmod(a0.x, c.v[limb], pc.q), addmod(a0.y, c.v[limb], pc.q)};
    auto product = [&](u64 x, u64 y) { return mulmod_barrett(x, y, pc.q, pc.r1, pc.r0); };
    st2(out + bi * o_bs + o0, u64x2{product(a0.x, s.x), product(a0.y, s.y)});
    st2(out + bi * o_bs + o1, u64x2{product(a1.x, addmod(a0.x, s.x, pc.q)), product(a1.y, addmod(a0.y, s.y, pc.q))});
    st2(out + bi * o_bs + o2, u64x2{product(a1.x, a1.x), product(a1.y, a1.y)});
}

hipError_t launch_square_linear(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int limbs, u64 n_batch, u64 a_bs,
                                u64 o_bs, int log_n, hipStream_t st) {
    if (t_analysis) {
        TALLY(mul, HISA_OP_MUL, n_batch, limbs);
        if (consts) {
            TALLY(mul_scalar, HISA_OP_MUL_SCALAR, n_batch, limbs);
            TALLY(add, HISA_OP_ADD, n_batch, limbs);
        }
    }
    DRY_RUN_RETURN();
    LimbConsts c = {};
    for (int i = 0; i < limbs && consts; i++) c.v[i] = consts[i];
    dim3 grid(PAIR_BLOCKS(log_n), limbs, (unsigned)n_batch);
    ProfScope prof__("square_linear_kernel", st);
    hipLaunchKernelGGL(square_linear_kernel, grid, dim3(NT), 0, st, primes, a, out, c, limbs, a_bs, o_bs, log_n);
    return hipGetLastError();
}

// ---- encryption profile -----------------------------------------------------
// ct[b] = (-a*s + e + m, a): a already sits in ct[b][1] (NTT form), e[b][limbs][N] in NTT form
__global__ __launch_bounds__(NT) void encrypt_combine_kernel(const PrimeConst* primes, const u64* secret, const u64* pt,
                                                             const u64* e, u64* ct, int limbs, u64 pt_bs, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 bi = blockIdx.z;
    const PrimeConst pc = primes[limb];
    const u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    const u64 off = (u64)limb * n + j;
    u64* c = ct + bi * 2 * limbs * n;
    u64 as = mulmod_barrett(c[(u64)limbs * n + off], secret[off], pc.q, pc.r1, pc.r0);
    u64 v = addmod(negmod(as, pc.q), e[bi * limbs * n + off], pc.q);
    c[off] = addmod(v, pt[bi * pt_bs + off], pc.q);
}

hipError_t launch_encrypt_combine(const PrimeConst* primes, const u64* secret, const u64* pt, const u64* e, u64* ct,
                                  int limbs, u64 n_batch, u64 pt_bs, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    dim3 grid((1u << log_n) / NT, limbs, (unsigned)n_batch);
    ProfScope prof__("encrypt_combine_kernel", st);
    hipLaunchKernelGGL(encrypt_combine_kernel, grid, dim3(NT), 0, st, primes, secret, pt, e, ct, limbs, pt_bs, log_n);
    return hipGetLastError();
}

// pt = c0 + c1*s (+ c2*s^2)
__global__ __launch_bounds__(NT) void decrypt_kernel(const PrimeConst* primes, const u64* secret, const u64* ct, u64 ct_bs, u64* pt,
                                                     int limbs, int polys, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    ct += (u64)blockIdx.z * ct_bs;
    pt += (u64)blockIdx.z * limbs * n;
    const PrimeConst pc = primes[limb];
    const u64 off = (u64)limb * n + (u64)blockIdx.x * NT + threadIdx.x;
    const u64 s = secret[off];
    u64 acc = ct[off], sp = s;
    for (int p = 1; p < polys; p++) {
        acc = addmod(acc, mulmod_barrett(ct[(u64)p * limbs * n + off], sp, pc.q, pc.r1, pc.r0), pc.q);
        sp = mulmod_barrett(sp, s, pc.q, pc.r1, pc.r0);
    }
    pt[off] = acc;
}

hipError_t launch_decrypt(const PrimeConst* primes, const u64* secret, const u64* ct, u64 ct_bs, u64* pt, int limbs, int polys,
                          u64 n_batch, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_batch == 0 || n_batch > 65535) return hipErrorInvalidValue;
    dim3 grid((1u << log_n) / NT, limbs, (unsigned)n_batch);
    ProfScope prof__("decrypt_kernel", st);
    hipLaunchKernelGGL(decrypt_kernel, grid, dim3(NT), 0, st, primes, secret, ct, ct_bs, pt, limbs, polys, log_n);
    return hipGetLastError();
}

// key digit: b = -a*s + e + [prime in digit] * (P mod q) * target ; a already in key_digit[1]
__global__ __launch_bounds__(NT) void key_combine_kernel(const PrimeConst* primes, const u64* secret, const u64* target,
                                                         const u64* e, const u64* pmod_all, u64* key_digit, int total,
                                                         int L, int alpha, int digit, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int prime = blockIdx.y;
    const PrimeConst pc = primes[prime];
    const u64 off = (u64)prime * n + (u64)blockIdx.x * NT + threadIdx.x;
    u64 a = key_digit[(u64)total * n + off];
    u64 v = addmod(negmod(mulmod_barrett(a, secret[off], pc.q, pc.r1, pc.r0), pc.q), e[off], pc.q);
    if (prime < L && prime / alpha == digit)
        v = addmod(v, mulmod_barrett(pmod_all[prime], target[off], pc.q, pc.r1, pc.r0), pc.q);
    key_digit[off] = v;
}

hipError_t launch_key_combine(const PrimeConst* primes, const u64* secret, const u64* target, const u64* e,
                              const u64* pmod_all, u64* key_digit, int total, int L, int alpha, int digit, int log_n,
                              hipStream_t st) {
    DRY_RUN_RETURN();
    dim3 grid((1u << log_n) / NT, total);
    ProfScope prof__("key_combine_kernel", st);
    hipLaunchKernelGGL(key_combine_kernel, grid, dim3(NT), 0, st, primes, secret, target, e, pmod_all, key_digit, total, L,
                       alpha, digit, log_n);
    return hipGetLastError();
}

// residues [n_rows][total][N] -> centred doubles in place, and back: what the fused key switch multiplies by is converted
// once per key instead of on every use
__global__ __launch_bounds__(NT) void key_to_doubles_kernel(const FpPrime* fprimes, u64* key, int log_n) {
    const FpPrime f = fprimes[blockIdx.y];
    const u64 off = (((u64)blockIdx.z * gridDim.y + blockIdx.y) << log_n) + (u64)blockIdx.x * NT + threadIdx.x;
    key[off] = (u64)__double_as_longlong(fp_centred_from_u64(key[off], f.p, f.half));
}

__global__ __launch_bounds__(NT) void key_to_residues_kernel(const FpPrime* fprimes, const u64* key, u64* out, int log_n) {
    const FpPrime f = fprimes[blockIdx.y];
    const u64 off = (((u64)blockIdx.z * gridDim.y + blockIdx.y) << log_n) + (u64)blockIdx.x * NT + threadIdx.x;
    out[off] = fp_canonical(__longlong_as_double((long long)key[off]), f.p, f.pinv);
}

hipError_t launch_key_to_doubles(const FpPrime* fprimes, u64* key, int n_rows, int total, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    ProfScope prof__("key_to_doubles_kernel", st);
    hipLaunchKernelGGL(key_to_doubles_kernel, dim3((1u << log_n) / NT, total, n_rows), dim3(NT), 0, st, fprimes, key, log_n);
    return hipGetLastError();
}

hipError_t launch_key_to_residues(const FpPrime* fprimes, const u64* key, u64* out, int n_rows, int total, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    ProfScope prof__("key_to_residues_kernel", st);
    hipLaunchKernelGGL(key_to_residues_kernel, dim3((1u << log_n) / NT, total, n_rows), dim3(NT), 0, st, fprimes, key, out, log_n);
    return hipGetLastError();
}

__global__ __launch_bounds__(NT) void square_kernel(const PrimeConst* primes, const u64* s, u64* out, int log_n) {
    const u64 n = (u64)1 << log_n;
    const PrimeConst pc = primes[blockIdx.y];
    const u64 off = (u64)blockIdx.y * n + (u64)blockIdx.x * NT + threadIdx.x;
    out[off] = mulmod_barrett(s[off], s[off], pc.q, pc.r1, pc.r0);
}

hipError_t launch_pointwise_square(const PrimeConst* primes, const u64* s, u64* out, int total, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    dim3 grid((1u << log_n) / NT, total);
    ProfScope prof__("square_kernel", st);
    hipLaunchKernelGGL(square_kernel, grid, dim3(NT), 0, st, primes, s, out, log_n);
    return hipGetLastError();
}

// sigma_g in NTT form is a pure gather: out[i] = in[src(i)] with
// 2*bitrev(src)+1 = (2*bitrev(i)+1)*g mod 2N.  Aligned blocks map to aligned blocks.
__global__ __launch_bounds__(NT) void automorph_ntt_kernel(const u64* in, u64 in_bs, u64* out, u64 out_bs, u64 g,
                                                           int log_n) {
    const u64 n = (u64)1 << log_n;
    const uint32_t i = blockIdx.x * NT + threadIdx.x;
    const uint32_t mask = (2u << log_n) - 1;
    uint32_t e = 2 * (__brev(i) >> (32 - log_n)) + 1;
    uint32_t e2 = (uint32_t)((u64)e * g) & mask;
    uint32_t src = __brev((e2 - 1) >> 1) >> (32 - log_n);
    out[(u64)blockIdx.z * out_bs + (u64)blockIdx.y * n + i] = in[(u64)blockIdx.z * in_bs + (u64)blockIdx.y * n + src];
}

hipError_t launch_automorph_ntt(const u64* in, u64 in_bs, u64* out, u64 out_bs, u64 galois, int n_polys, u64 n_batch,
                                int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    dim3 grid((1u << log_n) / NT, n_polys, (unsigned)n_batch);
    ProfScope prof__("automorph_ntt_kernel", st);
    hipLaunchKernelGGL(automorph_ntt_kernel, grid, dim3(NT), 0, st, in, in_bs, out, out_bs, galois, log_n);
    return hipGetLastError();
}

// The same gather for several automorphisms of the same n_batch inputs in one launch: blockIdx.z = s * n_batch + b,
// out entry (s, b) = sigma_{g[s]}(in entry b).
__global__ __launch_bounds__(NT) void automorph_steps_kernel(const u64* in, u64 in_bs, u64* out, u64 out_bs, GaloisTab tab,
                                                             unsigned n_batch, int log_n) {
    const u64 n = (u64)1 << log_n;
    const uint32_t i = blockIdx.x * NT + threadIdx.x;
    const uint32_t mask = (2u << log_n) - 1;
    const unsigned s = blockIdx.z / n_batch, b = blockIdx.z % n_batch;
    uint32_t e = 2 * (__brev(i) >> (32 - log_n)) + 1;
    uint32_t e2 = (uint32_t)((u64)e * tab.g[s]) & mask;
    uint32_t src = __brev((e2 - 1) >> 1) >> (32 - log_n);
    out[(u64)blockIdx.z * out_bs + (u64)blockIdx.y * n + i] = in[(u64)b * in_bs + (u64)blockIdx.y * n + src];
}

hipError_t launch_automorph_steps(const u64* in, u64 in_bs, u64* out, u64 out_bs, const GaloisTab& tab, int n_steps,
                                  int n_polys, u64 n_batch, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_steps < 1 || n_steps > GALOIS_TAB_MAX || n_batch == 0 || (u64)n_steps * n_batch > 65535) return hipErrorInvalidValue;
    for (int s = 0; s < n_steps; s++)
        if (tab.g[s] == 0) return hipErrorInvalidValue;
    dim3 grid((1u << log_n) / NT, n_polys, (unsigned)(n_steps * n_batch));
    ProfScope prof__("automorph_steps_kernel", st);
    hipLaunchKernelGGL(automorph_steps_kernel, grid, dim3(NT), 0, st, in, in_bs, out, out_bs, tab, (unsigned)n_batch, log_n);
    return hipGetLastError();
}

// acc[b][poly] += P * add[b][poly] on the limbs of q_0 .. q_{l-1}, for the polynomials the addend has: what a
// ciphertext contributes to key-switch accumulators that are divided by P later.  acc entries are (ciphertext,
// polynomial) pairs acc_bs words apart; pmod[i] = P mod q_i.
__global__ __launch_bounds__(NT) void fold_addend_kernel(const PrimeConst* primes, u64* acc, u64 acc_bs, const u64* add, u64 add_bs,
                                                         u64 add_ps, int add_polys, const u64* pmod, int log_n) {
    const u64 n = (u64)1 << log_n;
    const int limb = blockIdx.y;
    const u64 e = blockIdx.z, ct = e >> 1;
    const int poly = (int)(e & 1);
    if (poly >= add_polys) return;
    const PrimeConst pc = primes[limb];
    const u64 j = (u64)limb * n + pair_at(), pm = pmod[limb];
    u64* dst = acc + e * acc_bs + j;
    const u64x2 v = ld2(add + ct * add_bs + (u64)poly * add_ps + j), x = ld2(dst);
    st2(dst, u64x2{addmod(x.x, mulmod_barrett(v.x, pm, pc.q, pc.r1, pc.r0), pc.q), addmod(x.y, mulmod_barrett(v.y, pm, pc.q, pc.r1, pc.r0), pc.q)});
}

hipError_t launch_fold_addend(const PrimeConst* primes, u64* acc, u64 acc_bs, const u64* add, u64 add_bs, u64 add_ps,
                              int add_polys, const u64* pmod, u64 n_cts, int l, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    const u64 n = (u64)1 << log_n;
    if (!primes || !acc || !add || !pmod || n_cts == 0 || 2 * n_cts > 65535 || l < 1 || add_polys < 1 || add_polys > 2)
        return hipErrorInvalidValue;
    if (acc_bs < (u64)l * n || add_ps < (u64)l * n || add_bs < (u64)add_polys * l * n) return hipErrorInvalidValue;
    dim3 grid(PAIR_BLOCKS(log_n), l, (unsigned)(2 * n_cts));
    ProfScope prof__("fold_addend_kernel", st);
    hipLaunchKernelGGL(fold_addend_kernel, grid, dim3(NT), 0, st, primes, acc, acc_bs, add, add_bs, add_ps, add_polys, pmod, log_n);
    return hipGetLastError();
}

// signed integer coefficients [n_pts][N] -> residues modulo primes[0..limbs-1] at out[p][0..limbs-1][N], the entries of
// out being out_limbs limbs apart
__global__ __launch_bounds__(NT) void reduce_i64_kernel(const PrimeConst* primes, const i64* coeffs, u64* out, int out_limbs,
                                                        int log_n) {
    const u64 n = (u64)1 << log_n;
    const PrimeConst pc = primes[blockIdx.y];
    const u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    const u64 p = blockIdx.z;
    i64 v = coeffs[p * n + j];
    u64 mag = v < 0 ? (u64)0 - (u64)v : (u64)v;
    u64 r = barrett128(0, mag, pc.q, pc.r1, pc.r0);
    out[(p * out_limbs + blockIdx.y) * n + j] = v < 0 ? negmod(r, pc.q) : r;
}

hipError_t launch_reduce_i64(const PrimeConst* primes, const i64* coeffs, u64* out, int limbs, int n_pts, int log_n,
                             hipStream_t st) {
    return launch_reduce_i64(primes, coeffs, out, limbs, limbs, n_pts, log_n, st);
}

hipError_t launch_reduce_i64(const PrimeConst* primes, const i64* coeffs, u64* out, int limbs, int out_limbs, int n_pts,
                             int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_pts <= 0 || limbs <= 0) return hipSuccess;
    dim3 grid((1u << log_n) / NT, limbs, n_pts);
    ProfScope prof__("reduce_i64_kernel", st);
    hipLaunchKernelGGL(reduce_i64_kernel, grid, dim3(NT), 0, st, primes, coeffs, out, out_limbs, log_n);
    return hipGetLastError();
}
