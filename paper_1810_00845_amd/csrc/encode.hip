// encode / decode in fp64 (the HEAAN-style packing of N/2 complex slots, slot
// j at the root exp(i*pi*5^j/N)), and the centred CRT lift that turns RNS
// coefficients into doubles.  Direct sums with exact integer angle reduction
// into a table of the 2N-th roots of unity.
#include "hisa_internal.hpp"
#include "modarith.hpp"
#include "fparith.hpp"

#define NT 256

// coeffs[p][k] = round( factor * sum_j re[p][j] cos(pi e/N) ),  e = g[j] k mod 2N, g[j] = 5^(slot of entry j) mod 2N.  One
// launch encodes n_pts real vectors that share the slot list g[count].  A real vector's coefficient N - k is minus
// coefficient k (g[j] is odd): both come from one sum, so that the residues in NTT form mirror each other exactly.
__global__ __launch_bounds__(NT) void encode_kernel(const double* cs, const uint32_t* g, const double* re, int count, double factor,
                                                    i64* coeffs, int log_n) {
    const uint32_t k = blockIdx.x * NT + threadIdx.x;     // < N / 2
    const uint32_t mask = (2u << log_n) - 1;
    const size_t p = blockIdx.y;
    const double* r = re + p * count;
    double acc = 0.0;
    for (int j = 0; j < count; j++) acc += r[j] * cs[(g[j] * k) & mask];
    const i64 v = (i64)round(acc * factor);
    i64* out = coeffs + (p << log_n);
    out[k] = v;
    out[k ? (1u << log_n) - k : 1u << (log_n - 1)] = k ? -v : 0;
}

hipError_t launch_encode(const double* cs, const uint32_t* g, const double* re, int count, int n_pts, double factor, i64* coeffs,
                         int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_pts <= 0) return hipSuccess;
    ProfScope prof__("encode_kernel", st);
    hipLaunchKernelGGL(encode_kernel, dim3((1u << log_n) / 2 / NT, n_pts), dim3(NT), 0, st, cs, g, re, count, factor, coeffs, log_n);
    return hipGetLastError();
}

// Plaintexts that are piecewise constant -- value v[p][b] on slot set S_b, zero elsewhere -- are linear combinations of
// the nb encodings of the indicator vectors of the S_b: coeffs[p][k] = round(factor * sum_b v[p][b] basis[b][k]) with
// basis[b][k] = sum_{j in S_b} cos(pi g_j k / N), which costs nb terms per coefficient instead of one per slot.  The second
// half of a basis row is minus the first read backwards, exactly, and so is every combination.
__global__ __launch_bounds__(NT) void encode_basis_kernel(const double* cs, const uint32_t* g, const int* set_begin,
                                                          double* basis, int log_n) {
    const uint32_t k = blockIdx.x * NT + threadIdx.x;     // < N / 2
    const uint32_t mask = (2u << log_n) - 1;
    const int b = blockIdx.y;
    double acc = 0.0;
    for (int j = set_begin[b]; j < set_begin[b + 1]; j++) acc += cs[(g[j] * k) & mask];
    double* row = basis + ((size_t)b << log_n);
    row[k] = acc;
    row[k ? (1u << log_n) - k : 1u << (log_n - 1)] = k ? -acc : 0.0;
}

__global__ __launch_bounds__(NT) void encode_combine_kernel(const double* basis, int nb, const double* v, double factor,
                                                            i64* coeffs, int log_n) {
    const uint32_t k = blockIdx.x * NT + threadIdx.x;
    const size_t p = blockIdx.y;
    double acc = 0.0;
    for (int b = 0; b < nb; b++) acc += v[p * nb + b] * basis[((size_t)b << log_n) + k];
    coeffs[(p << log_n) + k] = (i64)round(acc * factor);
}

hipError_t launch_encode_basis(const double* cs, const uint32_t* g, const int* set_begin, int nb, double* basis, int log_n,
                               hipStream_t st) {
    DRY_RUN_RETURN();
    if (nb <= 0) return hipSuccess;
    ProfScope prof__("encode_basis_kernel", st);
    hipLaunchKernelGGL(encode_basis_kernel, dim3((1u << log_n) / 2 / NT, nb), dim3(NT), 0, st, cs, g, set_begin, basis, log_n);
    return hipGetLastError();
}

hipError_t launch_encode_combine(const double* basis, int nb, const double* v, int n_pts, double factor, i64* coeffs,
                                 int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_pts <= 0) return hipSuccess;
    ProfScope prof__("encode_combine_kernel", st);
    hipLaunchKernelGGL(encode_combine_kernel, dim3((1u << log_n) / NT, n_pts), dim3(NT), 0, st, basis, nb, v, factor, coeffs,
                       log_n);
    return hipGetLastError();
}

// Centred mixed-radix digits v_i in (-q_i/2, q_i/2] with x = v_0 + q_0 (v_1 + q_1 (v_2 + ...)), then Horner in fp64.
// Small centred values have zero top digits, so the float result is accurate for them.  One launch lifts n_pts vectors
// [vec][limbs][N].
__global__ __launch_bounds__(NT) void crt_to_double_kernel(const PrimeConst* primes, const u64* x, int limbs,
                                                           const u64* ginv, const u64* ginv_sh, int L, double inv_scale,
                                                           double* out, int log_n) {
    const u64 n = (u64)1 << log_n;
    const u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    x += (u64)blockIdx.y * limbs * n;
    double val = 0.0;
    // digits are produced low to high; accumulate v_i * (q_0...q_{i-1}) in fp64 from the low end would lose the
    // small terms, so keep the digits and run Horner from the top
    i64 dig[HISA_MAX_Q];
    for (int i = 0; i < limbs; i++) {
        const PrimeConst qi = primes[i];
        u64 t = x[(u64)i * n + j];
        for (int m = 0; m < i; m++) {
            i64 vm = dig[m];
            u64 mag = vm < 0 ? (u64)(-vm) : (u64)vm;
            u64 r = barrett128(0, mag, qi.q, qi.r1, qi.r0);
            if (vm < 0) r = negmod(r, qi.q);
            t = submod(t, r, qi.q);
            t = shoup_mul(t, ginv[(u64)m * L + i], ginv_sh[(u64)m * L + i], qi.q);
        }
        dig[i] = t > qi.half ? (i64)t - (i64)qi.q : (i64)t;
    }
    for (int i = limbs - 1; i >= 0; i--) val = val * (double)primes[i].q + (double)dig[i];
    out[(u64)blockIdx.y * n + j] = val * inv_scale;
}

hipError_t launch_crt_to_double(const PrimeConst* primes, const u64* coeff_form, int limbs, const u64* garner_inv,
                                const u64* garner_inv_sh, int L, double inv_scale, double* out, int n_pts, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_pts < 1 || n_pts > 65535) return hipErrorInvalidValue;
    ProfScope prof__("crt_to_double_kernel", st);
    hipLaunchKernelGGL(crt_to_double_kernel, dim3((1u << log_n) / NT, n_pts), dim3(NT), 0, st, primes, coeff_form, limbs,
                       garner_inv, garner_inv_sh, L, inv_scale, out, log_n);
    return hipGetLastError();
}

// The same lift for primes below 2^50 from centred doubles, the digits in registers (MAXL bounds the limbs): a step of the
// digit recurrence is a difference and one exact product instead of three 64-bit integer ones and a local array.
// N = 2^14, 12 limbs: 4 us a vector against 15.
template <int MAXL>
__global__ __launch_bounds__(NT) void crt_fp_kernel(const FpPrime* primes, const double* x, int limbs, const double* ginv, int L,
                                                    double inv_scale, double* out, int log_n) {
    const u64 n = (u64)1 << log_n;
    const u64 j = (u64)blockIdx.x * NT + threadIdx.x;
    x += (u64)blockIdx.y * limbs * n;
    double dig[MAXL];
#pragma unroll
    for (int i = 0; i < MAXL; i++) dig[i] = i < limbs ? x[(u64)i * n + j] : 0.0;
#pragma unroll
    for (int i = 1; i < MAXL; i++) {
        if (i < limbs) {
            const double p = primes[i].p, pinv = primes[i].pinv;
            double t = dig[i];
#pragma unroll
            for (int m = 0; m < i; m++) t = fp_mulmod(t - dig[m], ginv[(u64)m * L + i], p, pinv);
            dig[i] = fp_norm(t, p, pinv);
        }
    }
    double val = 0.0;
#pragma unroll
    for (int i = MAXL - 1; i >= 0; i--)
        if (i < limbs) val = val * primes[i].p + dig[i];
    out[(u64)blockIdx.y * n + j] = val * inv_scale;
}

hipError_t launch_crt_fp(const FpPrime* fprimes, const double* centred, int limbs, const double* garner_inv, int L, double inv_scale,
                         double* out, int n_pts, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (!fprimes || !centred || !garner_inv || !out || limbs < 1 || n_pts < 1 || n_pts > 65535) return hipErrorInvalidValue;
    ProfScope prof__("crt_fp_kernel", st);
    const dim3 grid((1u << log_n) / NT, n_pts);
    if (limbs <= 4) hipLaunchKernelGGL(crt_fp_kernel<4>, grid, dim3(NT), 0, st, fprimes, centred, limbs, garner_inv, L, inv_scale, out, log_n);
    else if (limbs <= 8) hipLaunchKernelGGL(crt_fp_kernel<8>, grid, dim3(NT), 0, st, fprimes, centred, limbs, garner_inv, L, inv_scale, out, log_n);
    else if (limbs <= 16) hipLaunchKernelGGL(crt_fp_kernel<16>, grid, dim3(NT), 0, st, fprimes, centred, limbs, garner_inv, L, inv_scale, out, log_n);
    else if (limbs <= 24) hipLaunchKernelGGL(crt_fp_kernel<24>, grid, dim3(NT), 0, st, fprimes, centred, limbs, garner_inv, L, inv_scale, out, log_n);
    else if (limbs <= HISA_MAX_Q) hipLaunchKernelGGL(crt_fp_kernel<HISA_MAX_Q>, grid, dim3(NT), 0, st, fprimes, centred, limbs, garner_inv, L, inv_scale, out, log_n);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// z_j = sum_k m_k exp(i*pi*e/N),  e = 5^j k mod 2N, for a handful of slots.  One workgroup per (slot, vector): thread t sums
// the coefficients k = t, t + DEC_NT, ..., then the partial sums are added pairwise (fixed order: reruns give the same
// bits).  z[vec][count] may be pinned host memory.
#define DEC_NT 1024
__global__ __launch_bounds__(DEC_NT) void decode_kernel(const double* cs, const double* sn, const double* m, int count, double2* z,
                                                        int log_n) {
    __shared__ double sr[DEC_NT], si[DEC_NT];
    const int j = blockIdx.x;
    const uint32_t n = 1u << log_n, mask = 2 * n - 1;
    m += (u64)blockIdx.y << log_n;
    // 5^j mod 2N by square and multiply
    uint32_t g = 1, base = 5, ex = (uint32_t)j;
    while (ex) {
        if (ex & 1) g = (g * base) & mask;
        base = (base * base) & mask;
        ex >>= 1;
    }
    double ar = 0.0, ai = 0.0;
    for (uint32_t k = threadIdx.x; k < n; k += DEC_NT) {
        const uint32_t e = (g * k) & mask;
        const double v = m[k];
        ar += v * cs[e];
        ai += v * sn[e];
    }
    sr[threadIdx.x] = ar; si[threadIdx.x] = ai;
    __syncthreads();
    for (int h = DEC_NT / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) { sr[threadIdx.x] += sr[threadIdx.x + h]; si[threadIdx.x] += si[threadIdx.x + h]; }
        __syncthreads();
    }
    if (threadIdx.x == 0) z[(u64)blockIdx.y * count + j] = make_double2(sr[0], si[0]);
}

hipError_t launch_decode(const double* cs, const double* sn, const double* m, int count, int n_pts, void* z, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (count <= 0) return hipSuccess;
    if (n_pts < 1 || n_pts > 65535) return hipErrorInvalidValue;
    ProfScope prof__("decode_kernel", st);
    hipLaunchKernelGGL(decode_kernel, dim3(count, n_pts), dim3(DEC_NT), 0, st, cs, sn, m, count, (double2*)z, log_n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The same two maps in O(N log N): the "special" FFT over the slot order 5^j
// ---------------------------------------------------------------------------
// With u_k = m_k + i m_{k+n} (n = N/2) the slot values are z_j = sum_{k<n} u_k zeta_j^k, zeta_j = exp(i pi 5^j / N).
// Splitting k into even and odd halves the problem: zeta_j^2 are the slot roots of the ring of half the degree,
// zeta_{j+n/2} = -zeta_j (5^(n/2) = N + 1 mod 2N), so
//     z_j = E_j + zeta_j O_j,   z_{j+n/2} = E_j - zeta_j O_j   (j < n/2),
// a radix-2 decimation-in-time transform from bit-reversed input whose stage of length `len` uses the twiddles
// exp(i pi (5^j mod 4 len) / (2 len)), j < len/2, read from the table of 2N-th roots.  The matrix (zeta_j^k) is
// unitary up to the factor n, so the inverse (encode) runs the stages backwards with conjugate twiddles.
// Stages up to SF_C = 1024 points run in LDS, one workgroup per chunk of consecutive points, two stages per exchange;
// the longer ones (at most five) take one launch together, a thread holding the points 1024 apart that they connect, and
// that launch also is the end at the slots: it reads the values to encode, or writes the decoded ones, straight from or to
// pinned host memory.  Twiddles come from a table in stage order (entry half + j: stage of length 2 half), which
// neighbouring threads read side by side; all of a chunk's are fetched before its first exchange.
// A vector at N = 2^14: two launches of 4-5 us each way; one launch per long stage and twiddles gathered from the
// table of roots through 5^j took 35 us.
#define SF_C 1024
#define SF_LOGC 10
#define SF_T 256
#define SF_LT 64      // threads of a workgroup of the long stages: up to 64 values each, and few of them
typedef double2 cplx;

__device__ __forceinline__ cplx sf_mul(cplx a, cplx b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ cplx sf_mulc(cplx a, cplx b) { return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y); }   // a * conj(b)
__device__ __forceinline__ cplx sf_add(cplx a, cplx b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ cplx sf_sub(cplx a, cplx b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ int sf_pad(int i) { return i + (i >> 3); }    // 16-byte elements: spreads strides of 4, 16, .. over the banks

// The end of an encoding: u_k = m_k + i m_{k+n} times factor, rounded.  mirror (real slot values): m_{N-k} = -m_k is taken from
// the real part of u_k instead of the imaginary part of u_{n-k}, so that it holds exactly.
__device__ __forceinline__ void store_coeffs(i64* m, uint32_t k, uint32_t n, cplx u, double factor, bool mirror) {
    const i64 v = (i64)round(u.x * factor);
    m[k] = v;
    if (!mirror) m[k + n] = (i64)round(u.y * factor);
    else m[k ? 2 * n - k : n] = k ? -v : 0;
}

// stages of length 2 .. 1024 of one chunk per workgroup.  DECODE: from the coefficients m[vec][N], bit-reversed, to
// work[vec][n].  Else from work[vec][n] to coefficients k and k + n of the bit-reversed position, times factor, rounded
// (store_coeffs).
template <bool DECODE>
__global__ __launch_bounds__(SF_T) void sfft_local_kernel(const cplx* tw, const double* m, cplx* work, double factor, i64* coeffs,
                                                          int log_n, bool mirror) {
    __shared__ cplx buf[SF_C + SF_C / 8];
    const uint32_t n = 1u << (log_n - 1), base = blockIdx.x * SF_C, t = threadIdx.x;
    const size_t vec = blockIdx.y;
    cplx w1[5], w2[5], w3[5], x[4];
#pragma unroll
    for (int p = 0; p < 5; p++) {           // stages of length 2 h and 4 h, h = 4^p
        const uint32_t h = 1u << (2 * p), j = t & (h - 1);
        w1[p] = tw[h + j]; w2[p] = tw[2 * h + j]; w3[p] = tw[3 * h + j];
    }
    if (DECODE) {
        const double* mv = m + (vec << log_n);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t src = __brev(base + 4 * t + i) >> (32 - (log_n - 1));
            x[i] = make_double2(mv[src], mv[src + n]);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; i++) x[i] = work[vec * n + base + t + 256 * i];
    }
#pragma unroll
    for (int q = 0; q < 5; q++) {
        const int p = DECODE ? q : 4 - q;
        const uint32_t h = 1u << (2 * p), j = t & (h - 1), at = ((t - j) << 2) + j;
        if (q) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 4; i++) x[i] = buf[sf_pad(at + h * i)];     // and written back to the same places below
        }
        if (DECODE) {
            const cplx b = sf_mul(x[1], w1[p]), d = sf_mul(x[3], w1[p]);
            const cplx a0 = sf_add(x[0], b), a1 = sf_sub(x[0], b), c0 = sf_mul(sf_add(x[2], d), w2[p]), c1 = sf_mul(sf_sub(x[2], d), w3[p]);
            x[0] = sf_add(a0, c0); x[2] = sf_sub(a0, c0); x[1] = sf_add(a1, c1); x[3] = sf_sub(a1, c1);
        } else {
            const cplx a0 = sf_add(x[0], x[2]), c0 = sf_mulc(sf_sub(x[0], x[2]), w2[p]);
            const cplx a1 = sf_add(x[1], x[3]), c1 = sf_mulc(sf_sub(x[1], x[3]), w3[p]);
            x[0] = sf_add(a0, a1); x[1] = sf_mulc(sf_sub(a0, a1), w1[p]);
            x[2] = sf_add(c0, c1); x[3] = sf_mulc(sf_sub(c0, c1), w1[p]);
        }
        if (q < 4) {
#pragma unroll
            for (int i = 0; i < 4; i++) buf[sf_pad(at + h * i)] = x[i];
        }
    }
    if (DECODE) {
#pragma unroll
        for (int i = 0; i < 4; i++) work[vec * n + base + t + 256 * i] = x[i];
    } else {
        i64* cv = coeffs + (vec << log_n);
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const uint32_t k = __brev(base + 4 * t + i) >> (32 - (log_n - 1));
            store_coeffs(cv, k, n, x[i], factor, mirror);
        }
    }
}

// The S stages longer than 1024 points (n = 1024 2^S), a thread per residue modulo 1024.  DECODE: work[vec][n] -> the first
// `count` slots, z[vec][count].  Else slot values -> work[vec][n]: re/im[vec][count] at slots 0 .. count - 1 (im may be
// null), zeros behind them, or, re null, what work holds.
template <int S, bool DECODE>
__global__ __launch_bounds__(SF_LT) void sfft_long_kernel(const cplx* tw, cplx* work, const double* re, const double* im, int count,
                                                         cplx* z) {
    constexpr int P = 1 << S;
    constexpr uint32_t n = 1024u << S;
    const uint32_t r = blockIdx.x * SF_LT + threadIdx.x;
    const size_t vec = blockIdx.y;
    cplx x[P];
#pragma unroll
    for (int k = 0; k < P; k++) {
        const uint32_t pos = r + 1024u * k;
        if (DECODE || !re) x[k] = work[vec * n + pos];
        else x[k] = (int)pos < count ? make_double2(re[vec * count + pos], im ? im[vec * count + pos] : 0.0) : make_double2(0.0, 0.0);
    }
#pragma unroll
    for (int q = 0; q < S; q++) {
        const int s = DECODE ? q : S - 1 - q, bit = 1 << s;        // stage of length 2048 2^s
#pragma unroll
        for (int k = 0; k < P; k++) {
            if (k & bit) continue;
            const cplx w = tw[(1024u << s) + r + 1024u * (k & (bit - 1))];
            if (DECODE) {
                const cplx v = sf_mul(x[k | bit], w), u = x[k];
                x[k] = sf_add(u, v); x[k | bit] = sf_sub(u, v);
            } else {
                const cplx u = x[k], v = x[k | bit];
                x[k] = sf_add(u, v); x[k | bit] = sf_mulc(sf_sub(u, v), w);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < P; k++) {
        const uint32_t pos = r + 1024u * k;
        if (!DECODE) work[vec * n + pos] = x[k];
        else if ((int)pos < count) z[vec * count + pos] = x[k];
    }
}

template <bool DECODE>
static hipError_t launch_long(const cplx* tw, cplx* work, const double* re, const double* im, int count, cplx* z, int n_pts, int log_n,
                              hipStream_t st) {
    const dim3 grid(1024 / SF_LT, n_pts);
    switch (log_n) {
        case 11: hipLaunchKernelGGL((sfft_long_kernel<0, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        case 12: hipLaunchKernelGGL((sfft_long_kernel<1, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        case 13: hipLaunchKernelGGL((sfft_long_kernel<2, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        case 14: hipLaunchKernelGGL((sfft_long_kernel<3, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        case 15: hipLaunchKernelGGL((sfft_long_kernel<4, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        case 16: hipLaunchKernelGGL((sfft_long_kernel<5, DECODE>), grid, dim3(SF_LT), 0, st, tw, work, re, im, count, z); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// N = 2^10 only: all nine stages of its 512 points, one workgroup per vector, radix 2.  DECODE: m -> z; else re/im or work
// -> coeffs.
template <bool DECODE>
__global__ __launch_bounds__(SF_T) void sfft_small_kernel(const cplx* tw, const double* m, const cplx* work, const double* re,
                                                          const double* im, int count, cplx* z, double factor, i64* coeffs, bool mirror) {
    __shared__ cplx buf[512];
    const size_t vec = blockIdx.x;
    for (uint32_t r = threadIdx.x; r < 512; r += SF_T) {
        if (DECODE) {
            const uint32_t src = __brev(r) >> 23;
            buf[r] = make_double2(m[vec * 1024 + src], m[vec * 1024 + src + 512]);
        } else if (re) {
            buf[r] = (int)r < count ? make_double2(re[vec * count + r], im ? im[vec * count + r] : 0.0) : make_double2(0.0, 0.0);
        } else {
            buf[r] = work[vec * 512 + r];
        }
    }
    for (int s = 0; s < 9; s++) {
        const uint32_t half = 1u << (DECODE ? s : 8 - s), j = threadIdx.x & (half - 1), i0 = ((threadIdx.x - j) << 1) + j;
        const cplx w = tw[half + j];
        __syncthreads();
        const cplx u = buf[i0], v = buf[i0 + half];
        if (DECODE) {
            const cplx t = sf_mul(v, w);
            buf[i0] = sf_add(u, t); buf[i0 + half] = sf_sub(u, t);
        } else {
            buf[i0] = sf_add(u, v); buf[i0 + half] = sf_mulc(sf_sub(u, v), w);
        }
    }
    __syncthreads();
    for (uint32_t r = threadIdx.x; r < 512; r += SF_T) {
        if (DECODE) {
            if ((int)r < count) z[vec * count + r] = buf[r];
        } else {
            const uint32_t k = __brev(r) >> 23;
            store_coeffs(coeffs + vec * 1024, k, 512, buf[r], factor, mirror);
        }
    }
}

// encode direction, sparse input: count values per vector at the listed slots of work[vec][n], which the launcher cleared
__global__ __launch_bounds__(SF_T) void sfft_fill_kernel(const double* re, const double* im, const uint32_t* slots, int count,
                                                         cplx* work, int log_n) {
    const size_t vec = blockIdx.y;
    const int i = blockIdx.x * SF_T + threadIdx.x;
    if (i < count) work[(vec << (log_n - 1)) + slots[i]] = make_double2(re[vec * count + i], im ? im[vec * count + i] : 0.0);
}

// m[n_pts][N] -> z[n_pts][count] complex (may be pinned host memory); work: n_pts * n complex numbers
hipError_t launch_decode_fft(const void* tw, const double* m, int count, int n_pts, void* work, void* z, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (count <= 0 || n_pts <= 0) return hipSuccess;
    if (!tw || !m || !work || !z || log_n < 10 || log_n > 16 || count > (1 << (log_n - 1)) || n_pts > 65535) return hipErrorInvalidValue;
    const uint32_t n = 1u << (log_n - 1);
    ProfScope prof__("decode_fft", st);
    if (log_n == 10) {
        hipLaunchKernelGGL(sfft_small_kernel<true>, dim3(n_pts), dim3(SF_T), 0, st, (const cplx*)tw, m, nullptr, nullptr, nullptr, count,
                           (cplx*)z, 1.0, nullptr, false);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(sfft_local_kernel<true>, dim3(n / SF_C, n_pts), dim3(SF_T), 0, st, (const cplx*)tw, m, (cplx*)work, 1.0, nullptr, log_n, false);
    return launch_long<true>((const cplx*)tw, (cplx*)work, nullptr, nullptr, count, (cplx*)z, n_pts, log_n, st);
}

// n_pts slot vectors -> coeffs[n_pts][N] = round(factor * (inverse transform)); values re/im[n_pts][count] at slots
// 0 .. count-1 (slots null; may be pinned host memory) or at slots[count] (device); work: n_pts * n complex numbers; mirror:
// store_coeffs (im null)
hipError_t launch_encode_fft(const void* tw, const double* re, const double* im, const uint32_t* slots, int count, int n_pts,
                             double factor, void* work, i64* coeffs, int log_n, hipStream_t st, bool mirror) {
    DRY_RUN_RETURN();
    if (n_pts <= 0) return hipSuccess;
    if (!tw || (mirror && im) || (!re && count) || !work || !coeffs || log_n < 10 || log_n > 16 || count < 0 || count > (1 << (log_n - 1)) || n_pts > 65535)
        return hipErrorInvalidValue;
    const uint32_t n = 1u << (log_n - 1);
    ProfScope prof__("encode_fft", st);
    if (slots || count == 0) {
        hipError_t e = hipMemsetAsync(work, 0, (size_t)n_pts * n * sizeof(cplx), st);
        if (e != hipSuccess) return e;
        if (count) hipLaunchKernelGGL(sfft_fill_kernel, dim3((count + SF_T - 1) / SF_T, n_pts), dim3(SF_T), 0, st, re, im, slots, count, (cplx*)work, log_n);
        re = im = nullptr;
    }
    if (log_n == 10) {
        hipLaunchKernelGGL(sfft_small_kernel<false>, dim3(n_pts), dim3(SF_T), 0, st, (const cplx*)tw, nullptr, (const cplx*)work, re, im,
                           count, nullptr, factor, coeffs, mirror);
        return hipGetLastError();
    }
    hipError_t e = launch_long<false>((const cplx*)tw, (cplx*)work, re, im, count, nullptr, n_pts, log_n, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sfft_local_kernel<false>, dim3(n / SF_C, n_pts), dim3(SF_T), 0, st, (const cplx*)tw, nullptr, (cplx*)work, factor,
                       coeffs, log_n, mirror);
    return hipGetLastError();
}
