// Single-launch negacyclic NTT / inverse NTT for N = 2^12 .. 2^15 and primes
// below 2^50, with exact fp64 modular arithmetic (fparith.hpp), and the key
// inner products over several rotations.  (The transforms of key switching and
// rescale are in convert_fp.hip.)
//
// One workgroup transforms one limb-polynomial.  N/32 threads hold 32
// coefficients each in registers (the whole polynomial lives in the register
// file: at N = 2^15 one 1024-thread workgroup fills a CU's registers).  The log2 N
// butterfly levels run as three register-resident radix-32 phases; between
// phases the polynomial is transposed through LDS as two 32-bit halves, so the
// staging buffer is N*4 bytes plus padding (132 KiB at N = 2^15) and the transposes
// need no extra registers.  Global loads and stores are coalesced.
//
// Index bit fields of a coefficient index: idx = (a:5)(b:5)(c:K3), K3 = log2 N - 10
// (the four register mappings are listed at struct Geo).
// Forward (natural in, value at psi^(2 bitrev(i)+1) at index i out): decimation
// in time, levels 1..5 on a (mapping 1), 6..10 on b (2), 11.. on c (3), stores in
// mapping 4.  Inverse: the cyclic inverse transform as decimation in time from
// bit-reversed input (loads in mapping 4, levels on c in 3, then b in 2, then a
// in 1) followed by the untwist psi^-j / N.  Only the transpose 1 <-> 2 crosses waves (five workgroup barriers per
// transform); after it the waves run apart and overlap one another's LDS
// traffic, stores and next loads.
#include <cstdio>

#include "fp_device.hpp"

template <int K3>
struct Geo {
    static constexpr int LOGN = 10 + K3, TB = 5 + K3, THREADS = 1 << TB, N = 1 << LOGN, CM = (1 << K3) - 1;
    // A coefficient index is (a:5)(b:5)(c:K3), b = (b_high : 5-K3)(b_low : K3).  Four ways to spread the N coefficients
    // over THREADS threads x 32 registers; in each the index is (a term of the thread) | (a compile-time term of the
    // register) with disjoint bits, so addressing needs one register per mapping, not one per element:
    //   1  thread (b, c),      register a             loads/stores of the side whose phase works on a; phase on a
    //   2  thread (a, c),      register b             phase on b
    //   3  thread (a, b_low),  register (b_high, c)   phase on c (2^(5-K3) groups of 2^K3 registers)
    //   4  thread (wave w, lane), register r: index 2048 w + 64 r + lane     coalesced loads/stores
    // In mappings 2, 3 and 4 wave w holds exactly the coefficients [2048 w, 2048 (w+1)), so the transposes between
    // them stay inside a wave and need no workgroup barrier; only 1 <-> 2 crosses waves.
    template <int M> static __device__ __forceinline__ int thread_idx(int t) {
        if (M == 1) return t;
        if (M == 2) return ((t >> K3) << TB) | (t & CM);
        if (M == 3) return ((t >> K3) << TB) | ((t & CM) << K3);
        return ((t >> 6) << 11) | (t & 63);
    }
    template <int M> static constexpr int reg_idx(int r) {
        return M == 1 ? (r << TB) : (M == 2 ? (r << K3) : (M == 3 ? (((r >> K3) << (2 * K3)) | (r & CM)) : (r << 6)));
    }
    // LDS word address of index x: x plus pad words (x >> 5, and one more shift for the small rings) that spread the
    // strided accesses of the mappings over the banks (conflict-free at N = 2^15, at most two-way below).  The
    // shifts act on disjoint bit fields, so the address of (thread | register) is the sum of the two addresses.
    static constexpr int PAD2 = K3 == 3 ? 7 : (K3 == 2 ? 8 : 0);
    static constexpr int LDS_WORDS = N + N / 32 + (PAD2 ? (N >> PAD2) : 0);
    static __device__ __forceinline__ constexpr int lds_of(int x) { return x + (x >> 5) + (PAD2 ? (x >> PAD2) : 0); }
    template <int M> static __device__ __forceinline__ int thread_lds(int t) { return lds_of(thread_idx<M>(t)); }
    template <int M> static constexpr int reg_lds(int r) { return lds_of(reg_idx<M>(r)); }
};

// transpose between two register mappings through LDS, 32-bit halves one after the other
template <int K3, int FROM, int TO, bool LOCAL = false>
__device__ __forceinline__ void exchange(double (&v)[32], uint32_t* lds, int t) {
    typedef Geo<K3> G;
    uint32_t* wr = lds + G::template thread_lds<FROM>(t);
    const uint32_t* rd = lds + G::template thread_lds<TO>(t);
    // the low words are dead once written, so the incoming low words take their registers: 64 live, not 96
    uint32_t lo[32], hi[32];
#pragma unroll
    for (int r = 0; r < 32; r++) { lo[r] = lo32(v[r]); hi[r] = hi32(v[r]); }
#pragma unroll
    for (int r = 0; r < 32; r++) wr[G::template reg_lds<FROM>(r)] = lo[r];
    xchg_sync<LOCAL>();
#pragma unroll
    for (int r = 0; r < 32; r++) lo[r] = rd[G::template reg_lds<TO>(r)];
    xchg_sync<LOCAL>();
#pragma unroll
    for (int r = 0; r < 32; r++) wr[G::template reg_lds<FROM>(r)] = hi[r];
    xchg_sync<LOCAL>();
#pragma unroll
    for (int r = 0; r < 32; r++) hi[r] = rd[G::template reg_lds<TO>(r)];
    xchg_sync<LOCAL>();
#pragma unroll
    for (int r = 0; r < 32; r++) v[r] = mk64(lo[r], hi[r]);
}

// Range: with centred twiddles (|w| <= 0.55 p after a factored product) a level takes max|v| = m p to at most
// (1.21 m + 0.5) p, so five levels from m = 1 (canonical input) stay below 6.2 p and from m = 0.5 (normalised)
// below 5.1 p, inside the 2^53 = 8 * 2^50 that exact integer arithmetic in doubles allows: one normalisation
// per phase is enough and none is needed inside a phase.
__device__ __forceinline__ void bfly(double& x, double& y, double w, double p, double pinv) {
    const double t = fp_mulmod(y, w, p, pinv);
    y = x - t;
    x = x + t;
}

// Twiddles.  The forward twiddle of level j of a phase factors as
//     psi^bitrev(((first + tpart) << j) + g)  =  psi^bitrev((first + tpart) << j)  *  psi^bitrev(g),
// a per-thread value (one per level: five loads per phase, stored at (first << j) + tpart so that lanes read
// consecutive addresses) times a value that is the same for every thread (the first entries of the table, read
// through the scalar cache).  The inverse twiddle psi^(-k N/m), k = (klow << kshift) + tlow, factors the same way.
// The per-thread values are fetched one phase ahead, before the transpose, so that their latency hides behind
// the LDS traffic; the products cost 26 modular multiplications per phase.
template <int BITS, int GROUPS>
__device__ __forceinline__ void load_fwd_tw(double (&bt)[GROUPS][5], rsrc_t tw, int first, const int (&tpart)[GROUPS]) {
#pragma unroll
    for (int grp = 0; grp < GROUPS; grp++)
#pragma unroll
        for (int j = 0; j < BITS; j++) bt[grp][j] = bloadf(tw, (uint32_t)tpart[grp] * 8u, (uint32_t)(first << j) * 8u);
}

// BITS levels over the register-index field of each group of 2^BITS registers (GROUPS groups), largest distance
// first.  UNIFORM: the twiddles depend on the register index only (first phase).
template <int BITS, int GROUPS, int STRIDE, bool UNIFORM>
__device__ __forceinline__ void fwd_phase(double (&v)[32], const double* tw, const double (&bt)[GROUPS][5], double p,
                                          double pinv) {
#pragma unroll
    for (int j = 0; j < BITS; j++) {
        const int half = BITS - 1 - j;
#pragma unroll
        for (int grp = 0; grp < GROUPS; grp++) {
#pragma unroll
            for (int g = 0; g < (1 << j); g++) {
                double w;
                if (UNIFORM) w = as_const(tw)[(1 << j) + g];
                else w = g == 0 ? bt[grp][j] : fp_mulmod(bt[grp][j], as_const(tw)[g], p, pinv);
#pragma unroll
                for (int lo = 0; lo < (1 << half); lo++) {
                    const int r0 = grp * STRIDE + ((g << (half + 1)) | lo);
                    bfly(v[r0], v[r0 + (1 << half)], w, p, pinv);
                }
            }
        }
    }
}

template <int BITS>
__device__ __forceinline__ void load_inv_tw(double (&bt)[5], rsrc_t utw, int t0, int tlow) {
#pragma unroll
    for (int j = 0; j < BITS; j++) bt[j] = bloadf(utw, (uint32_t)tlow * 8u, (8u << (t0 + j)));
}

// Inverse phase (decimation in time from bit-reversed input): level j pairs bit j of the field, smallest distance
// first; twiddle psi^(-k N/2^(t0+j)), k = (klow << t0) + tlow, klow = low j bits of the register field;
// = utw[2^(t0+j) + tlow] * utw[2^j + klow].  UNIFORM: t0 = 0, tlow = 0.
template <int BITS, int GROUPS, int STRIDE, bool UNIFORM>
__device__ __forceinline__ void inv_phase(double (&v)[32], const double* utw, const double (&bt)[5], double p, double pinv) {
#pragma unroll
    for (int j = 0; j < BITS; j++) {
#pragma unroll
        for (int klow = 0; klow < (1 << j); klow++) {
            // The very first level multiplies by 1.  (So does the first group of every later level of this phase, but
            // a butterfly without its product does not reduce y: the values would double per level and leave the
            // exact range after four of them.)
            const bool unit = UNIFORM && j == 0;
            double w = 1.0;
            if (UNIFORM) { if (!unit) w = as_const(utw)[(1 << j) + klow]; }
            else w = klow == 0 ? bt[j] : fp_mulmod(bt[j], as_const(utw)[(1 << j) + klow], p, pinv);
#pragma unroll
            for (int grp = 0; grp < GROUPS; grp++) {
#pragma unroll
                for (int hi = 0; hi < (1 << (BITS - 1 - j)); hi++) {
                    const int r0 = grp * STRIDE + ((hi << (j + 1)) | klow);
                    if (unit) {
                        const double x = v[r0], y = v[r0 + (1 << j)];
                        v[r0] = x + y;
                        v[r0 + (1 << j)] = x - y;
                    } else {
                        bfly(v[r0], v[r0 + (1 << j)], w, p, pinv);
                    }
                }
            }
        }
    }
}

// Second launch bound: waves per SIMD the register allocation must leave room for.  N = 2^15 needs 4 (one
// workgroup of 16 waves per CU, 128 registers).  At N = 2^14 the same cap lets two workgroups share a CU and
// overlap one's transposes with the other's arithmetic (measured 16% faster than one workgroup with 256
// registers); at N <= 2^13 the cap costs spills and the 256-register build is the faster one.
#ifndef NTT_FP_MIN_WAVES
#define NTT_FP_MIN_WAVES(K3) ((K3) >= 4 ? 4 : 2)
#endif
template <int K3, int MODE>
__global__ __launch_bounds__(Geo<K3>::THREADS, NTT_FP_MIN_WAVES(K3)) void ntt_fp_kernel(FpArgs a, FpTask tk) {
    typedef Geo<K3> G;
    extern __shared__ uint32_t lds[];
    const int t = threadIdx.x;
    // Persistent workgroups: each loops over its share of the tasks, so consecutive tasks on a CU run back to back
    // (no dispatch gap, the stores of one overlap the loads of the next).  Workgroups go to the eight XCDs
    // round-robin by id; each XCD gets a contiguous range of tasks, so that tasks sharing inputs (all target
    // limbs of one digit of one ciphertext) run on one XCD at about the same time and find them in its L2.
    const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, slots = gridDim.x >> 3;
    const int per_xcd = (a.n_tasks + 7) >> 3;
    const int task_end = min((xcd + 1) * per_xcd, a.n_tasks);
    constexpr bool INV = MODE == FP_INV_PLAIN;
    // limb-major, so that the compute units of an XCD work on one prime at a time and its twiddle tables (as much data as
    // the polynomial itself) stay in that L2
    const int n_entries = a.n_tasks / tk.period;
    for (int task = xcd * per_xcd + slot; task < task_end; task += slots) {
    const u64 b = task % n_entries;
    const int e = task / n_entries;
    const int pos = tk.pos[e], prime = tk.prime[e];
    const double p = as_const(&a.fprimes[prime].p)[0], pinv = as_const(&a.fprimes[prime].p)[1];
    // Global memory is touched in mapping 1 (lane <-> consecutive coefficients, register r a block of THREADS
    // further) on the side of the transform whose first/last phase works on the top bits, and in mapping 4 on the
    // other side, where the transposes stay inside a wave.
    constexpr int MIN = INV ? 4 : 1;    // mapping of the inverse transform's loads
    constexpr int MOUT = INV ? 1 : 4;   // mapping of the forward transform's stores
    const int t_in = G::template thread_idx<MIN>(t), t_out = G::template thread_idx<MOUT>(t);
    constexpr uint32_t LB = (uint32_t)G::N * 8u;   // bytes of one limb-polynomial
    const uint32_t t8 = (uint32_t)t * 8u, t8_in = (uint32_t)t_in * 8u, t8_out = (uint32_t)t_out * 8u;
    double v[32];

    // ---- load (mapping P1: lane <-> consecutive coefficients; register r holds coefficient r*THREADS + t) ----
    {
        const rsrc_t src = make_rsrc(a.in + b * a.in_bs + (u64)pos * G::N, LB);
#pragma unroll
        for (int r = 0; r < 32; r++) v[r] = fp_from_u64(bload(src, t8_in, (uint32_t)G::template reg_idx<MIN>(r) * 8u));
    }

    if (!INV) {
        const double* tw = a.ftw + (u64)prime * G::N;
        const rsrc_t twr = make_rsrc(tw, LB);
        double bt2[1][5];
        {   // levels 1..5 on a: twiddles depend on the register index only
            const double none[1][5] = {};
            fwd_phase<5, 1, 32, true>(v, tw, none, p, pinv);
        }
        {   // per-thread twiddles of levels 6..10 (index 2^(5+j) + a), fetched before the transpose
            const int tp[1] = {t >> K3};
            load_fwd_tw<5, 1>(bt2, twr, 32, tp);
            SCHED_FENCE();
        }
#pragma unroll
        for (int r = 0; r < 32; r++) v[r] = fp_norm(v[r], p, pinv);
        // the waves run apart between the wave-local transposes: all of them must have left the buffer before this
        // workgroup-wide transpose writes to it (its own last barrier guards the other direction)
        __syncthreads();
        exchange<K3, 1, 2>(v, lds, t);
        fwd_phase<5, 1, 32, false>(v, tw, bt2, p, pinv);
        constexpr int GROUPS = 1 << (5 - K3);
        double bt3[GROUPS][5];
        {   // levels 11.. on c: index 2^(10+j) + (a 32 + b), one group per b_high
            int tp[GROUPS];
#pragma unroll
            for (int grp = 0; grp < GROUPS; grp++) tp[grp] = ((t >> K3) << 5) | (grp << K3) | (t & G::CM);
            load_fwd_tw<K3, GROUPS>(bt3, twr, 1024, tp);
            SCHED_FENCE();
        }
#pragma unroll
        for (int r = 0; r < 32; r++) v[r] = fp_norm(v[r], p, pinv);
        exchange<K3, 2, 3, true>(v, lds, t);
        fwd_phase<K3, GROUPS, 1 << K3, false>(v, tw, bt3, p, pinv);
        exchange<K3, 3, MOUT, true>(v, lds, t);
    } else {
        const double* utw = a.utw + (u64)prime * G::N;
        const rsrc_t utwr = make_rsrc(utw, LB);
        double bt[5];
        exchange<K3, MIN, 3, true>(v, lds, t);
        {   // levels t = 0..K3-1 on c
            const double none[5] = {};
            inv_phase<K3, 1 << (5 - K3), 1 << K3, true>(v, utw, none, p, pinv);
        }
        load_inv_tw<5>(bt, utwr, K3, t & G::CM);   // levels K3 + j on b: k = (b mod 2^j) 2^K3 + c
        SCHED_FENCE();
#pragma unroll
        for (int r = 0; r < 32; r++) v[r] = fp_norm(v[r], p, pinv);
        exchange<K3, 3, 2, true>(v, lds, t);
        inv_phase<5, 1, 32, false>(v, utw, bt, p, pinv);
        load_inv_tw<5>(bt, utwr, G::TB, t);        // levels 5 + K3 + j on a: k = (a mod 2^j) 2^(5+K3) + (b, c)
        SCHED_FENCE();
#pragma unroll
        for (int r = 0; r < 32; r++) v[r] = fp_norm(v[r], p, pinv);
        __syncthreads();
        exchange<K3, 2, 1>(v, lds, t);
        inv_phase<5, 1, 32, false>(v, utw, bt, p, pinv);
    }

    const rsrc_t dst = make_rsrc(a.out + b * a.out_bs + (u64)pos * G::N, LB);
    if (!INV) {
#pragma unroll
        for (int r = 0; r < 32; r++)
            bstore(dst, t8_out, (uint32_t)G::template reg_idx<MOUT>(r) * 8u, fp_canonical(v[r], p, pinv));
    } else {
        const rsrc_t vtw = make_rsrc(a.vtw + (u64)prime * G::N, LB);
#pragma unroll
        for (int c = 0; c < 4; c++) {
            double w8[8];
            SCHED_FENCE();
#pragma unroll
            for (int k = 0; k < 8; k++) w8[k] = bloadf(vtw, t8, (uint32_t)((c * 8 + k) << G::TB) * 8u);
            SCHED_FENCE();
#pragma unroll
            for (int k = 0; k < 8; k++) {
                const int r = c * 8 + k;
                bstore(dst, t8, (uint32_t)(r << G::TB) * 8u, fp_canonical(fp_mulmod(v[r], w8[k], p, pinv), p, pinv));
            }
        }
    }
    }  // task loop
}

template <int K3, int MODE>
static hipError_t launch_one(const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st) {
    typedef Geo<K3> G;
    static bool attr_set = false;
    const size_t lds_bytes = (size_t)G::LDS_WORDS * 4;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute((const void*)ntt_fp_kernel<K3, MODE>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)lds_bytes);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    // the name rocprofv3 prints for this instantiation
    static char name[40] = "";
    if (!name[0]) snprintf(name, sizeof name, "ntt_fp_kernel<%d, %d>", K3, MODE);
    ProfScope prof__(name, st);
    FpArgs args = a;
    args.n_tasks = (int)(n_batch * tk.period);
    static int n_cu = 0;
    if (!n_cu) {
        hipDeviceProp_t prop;
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return hipErrorInvalidDevice;
        n_cu = prop.multiProcessorCount > 8 ? prop.multiProcessorCount : 8;
    }
    // as many workgroups as are resident on the chip at once
    static int per_cu = 0;
    if (!per_cu) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, (const void*)ntt_fp_kernel<K3, MODE>, G::THREADS, lds_bytes) != hipSuccess ||
            nb < 1)
            nb = 1;
        per_cu = nb;
    }
    unsigned grid = (unsigned)(n_cu * per_cu) & ~7u;
    const unsigned need = (unsigned)((args.n_tasks + 7) / 8) * 8;
    if (grid > need) grid = need;
    hipLaunchKernelGGL((ntt_fp_kernel<K3, MODE>), dim3(grid), dim3(G::THREADS), lds_bytes, st, args, tk);
    return hipGetLastError();
}

template <int MODE>
static hipError_t dispatch_k3(int log_n, const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st) {
    switch (log_n) {
        case 12: return launch_one<2, MODE>(a, tk, n_batch, st);
        case 13: return launch_one<3, MODE>(a, tk, n_batch, st);
        case 14: return launch_one<4, MODE>(a, tk, n_batch, st);
        case 15: return launch_one<5, MODE>(a, tk, n_batch, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ntt_fp(int mode, int log_n, const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_batch == 0 || tk.period <= 0) return hipSuccess;
    // every pointer a mode dereferences must be set: a missing one is a host error, not a device fault
    if (tk.period > HISA_MAX_PRIMES || !a.fprimes || !a.in || !a.out) return hipErrorInvalidValue;
    for (int e = 0; e < tk.period; e++)
        if (tk.prime[e] < 0) return hipErrorInvalidValue;
    if (mode == FP_FWD_PLAIN) return a.ftw ? dispatch_k3<FP_FWD_PLAIN>(log_n, a, tk, n_batch, st) : hipErrorInvalidValue;
    if (mode == FP_INV_PLAIN) return a.utw && a.vtw ? dispatch_k3<FP_INV_PLAIN>(log_n, a, tk, n_batch, st) : hipErrorInvalidValue;
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// inner product with the switching key, fp64
// ---------------------------------------------------------------------------
#define IPF_NT 256
#define IPF_MAXD 8
// Keys are centred doubles here (key_to_doubles_kernel).
// Several rotations of the same ciphertexts: blockIdx.z is the rotation; its key values stay in registers while the
// thread walks over the batch.  The extended digits come from the unrotated polynomial and are gathered through the
// rotation's automorphism like the own-digit limbs.
__global__ __launch_bounds__(IPF_NT) void inner_product_steps_fp_kernel(const FpPrime* fprimes, const double* ext, u64 ext_bs,
                                                                        int digits, int l, int K, int L, int alpha, IpSteps steps,
                                                                        int total, const u64* own_src, u64 own_bs, u64* acc,
                                                                        u64 acc_bs, u64 n_batch, const u64* c0_src,
                                                                        const u64* pmod, int log_n) {
    const u64 n = (u64)1 << log_n;
    const uint32_t j = blockIdx.x * IPF_NT + threadIdx.x;
    // the rotations of a limb run together: they read the same extended digits (through different automorphisms)
    const int x = blockIdx.z, s = blockIdx.y;
    const int ext_limbs = l + K;
    const int prime = x < l ? x : L + (x - l);
    const int own_digit = x < l ? x / alpha : -1;
    const double p = as_const(&fprimes[prime].p)[0], pinv = as_const(&fprimes[prime].p)[1];
    const u64* key = steps.key[s];
    const uint32_t jsrc = galois_src_fp(j, steps.galois[s], log_n);
    double kb[IPF_MAXD], ka[IPF_MAXD];
#pragma unroll
    for (int d = 0; d < IPF_MAXD; d++) {
        if (d < digits) {
            kb[d] = ((const double*)key)[(((u64)d * 2 + 0) * total + prime) * n + j];
            ka[d] = ((const double*)key)[(((u64)d * 2 + 1) * total + prime) * n + j];
        }
    }
    // c0_src: the first accumulator also takes P * sigma_s(c0) on the limbs of q (what ModDown turns back into
    // sigma_s(c0): the rotated ciphertext is then the ModDown of the accumulators alone)
    const bool fold = c0_src != nullptr && x < l;
    const double pm = fold ? fp_from_u64(pmod[prime]) : 0.0;
    for (u64 b = 0; b < n_batch; b++) {
        double sb = 0.0, sa = 0.0;
#pragma unroll
        for (int d = 0; d < IPF_MAXD; d++) {
            if (d < digits) {
                const double e = d == own_digit ? fp_from_u64(own_src[b * own_bs + (u64)x * n + jsrc])
                                                : ext[b * ext_bs + ((u64)d * ext_limbs + x) * n + jsrc];
                sb += fp_mulmod(e, kb[d], p, pinv);
                sa += fp_mulmod(e, ka[d], p, pinv);
            }
        }
        if (fold) sb = fp_norm(sb, p, pinv) + fp_mulmod(fp_from_u64(c0_src[b * own_bs + (u64)x * n + jsrc]), pm, p, pinv);
        u64* dst = acc + ((u64)s * n_batch + b) * acc_bs;
        dst[(u64)x * n + j] = fp_canonical(sb, p, pinv);
        dst[((u64)ext_limbs + x) * n + j] = fp_canonical(sa, p, pinv);
    }
}

// The sum over rotations, before the division by P: entry (s, b) of ext / own_src is term s of output b (its digits
// computed from the unrotated polynomial, gathered here through sigma_s like the own-digit limbs) -- or, with
// shared_input, entry b for every s: all terms of an output rotate the same ciphertext --
// acc[b] = sum_s sum_j sigma_s(e_{s,b,j}) * key_s[j], and on the limbs of q P times what needs no key: sum_s sigma_s(c0 of
// term s) and the two polynomials of `plain` (null: none).  P c divided by P is c again, and it leaves the special limbs
// alone: the division that follows needs no addend.
// A thread owns a coefficient of a limb and up to IPS_BCH outputs, for which a rotation's key values serve once loaded; the
// workgroups of a limb run together, so the key rows that each of them reads come from the L2 after the first.  GROUPS = 4: where
// workgroups are few, a thread would be a chain of up to 32 rounds of dependent loads; the four waves of a workgroup then take
// the same 64 coefficients and every fourth rotation each, and their sums meet in LDS.  ONCE: one group of outputs, keys that pass the
// caches by (STREAMED_KEY_BYTES; three digits, 28 limbs at N = 2^15 308 -> 296 us, 22 limbs 190 -> 164).
// Against sums in one chain a thread, a reduction a product, and c0 and addend in two launches of their own (us, all sums of a network):
// LeNet-small 203 -> 105, LeNet-medium 1095 -> 678, SqueezeNet-style 2087 -> 1758 (there the keys, 640 MB a launch of one output, bound
// it).  In one wave or over four, by workgroups of whole chains: 288 of them 40 -> 32 us a launch, 1792 50 -> 41, 2560 and more even.
// DIGITS: up to three are known to the compiler and a rotation's loads are one wait; more go one after the other.  (All of four
// to eight at once took 160 registers: 64 outputs of nine rotations at N = 2^13, 8 limbs, us: four digits 1618 against 1358, eight
// 2638 against 2292, with a reduction a product 1461 and 2392; one output at N = 2^15, 12 limbs, four digits 289, 215, 225.)
// Ranges: all factors within p / 2; the sums are reduced before they hold more terms than their plan allows.  At most eight rotations
// a wave add canonical c0 values when GROUPS = 4; otherwise those are normalised every sixth rotation, on top of a normalised
// value: 6.5 p < 2^53.
#define IPS_BCH 4
#define IPS_FEW 2048    // workgroups of whole chains
template <int GROUPS, int DIGITS, bool ONCE>
__device__ __forceinline__ void inner_product_sum(
    const FpPrime* fprimes, const double* ext, u64 ext_bs, int digits, int l, int K, int L, int alpha, const IpSteps& steps, int n_steps, int total,
    const u64* own_src, u64 own_bs, u64* acc, u64 acc_bs, u64 n_batch, int shared_input, const u64* c0_src, const u64* plain, u64 plain_bs,
    const u64* pmod, int log_n) {
    constexpr int COEFFS = IPF_NT / GROUPS, AT_ONCE = DIGITS ? DIGITS : 1;
    const u64 n = (u64)1 << log_n;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
    const uint32_t j = blockIdx.x * COEFFS + (GROUPS == 1 ? threadIdx.x : lane);
    const int x = blockIdx.z;      // the groups of outputs of a limb run together: they read the same key rows
    const u64 b0 = (u64)blockIdx.y * IPS_BCH;
    const int live = (int)(n_batch - b0 < IPS_BCH ? n_batch - b0 : IPS_BCH);
    const int ext_limbs = l + K;
    const int prime = x < l ? x : L + (x - l);
    const int own_digit = x < l ? x / alpha : -1;
    const double p = as_const(&fprimes[prime].p)[0], pinv = as_const(&fprimes[prime].p)[1];
    const FpSumPlan plan = fp_sum_plan(p);
    const int fold_every = plan.terms / digits;                  // rotations
    FpSum sb[IPS_BCH], sa[IPS_BCH];
    double tc[IPS_BCH];
#pragma unroll
    for (int u = 0; u < IPS_BCH; u++) { sb[u] = sa[u] = FpSum{plan.base, 0.0}; tc[u] = 0.0; }
    auto fold = [&](FpSum& s) { s = FpSum{plan.base, fp_norm(fp_sum_value(s, plan.base, p, pinv), p, pinv)}; };
    int pending = 0, c0_pending = 0;
    for (int s = GROUPS == 1 ? 0 : wave; s < n_steps; s += GROUPS) {
        const double* key = (const double*)steps.key[s] + (u64)prime * n + j;
        const uint32_t jsrc = galois_src_fp(j, steps.galois[s], log_n);
        const u64 entry0 = (shared_input ? 0 : (u64)s * n_batch) + b0;
        // a rotation's loads all together where the digits are known to the compiler: one wait
#pragma unroll 1
        for (int d0 = 0; d0 < (DIGITS ? DIGITS : digits); d0 += AT_ONCE) {
            double kb[AT_ONCE], ka[AT_ONCE], e[AT_ONCE][IPS_BCH], c0[IPS_BCH];
            const bool with_c0 = d0 == 0 && x < l;
#pragma unroll
            for (int i = 0; i < AT_ONCE; i++) {
                const int d = d0 + i;
                const double *key_b = key + (u64)(d * 2) * total * n, *key_a = key_b + (u64)total * n;
                kb[i] = ONCE ? __builtin_nontemporal_load(key_b) : *key_b;
                ka[i] = ONCE ? __builtin_nontemporal_load(key_a) : *key_a;
                const bool own = d == own_digit;
                const double* src = own ? (const double*)own_src + entry0 * own_bs + (u64)x * n + jsrc
                                        : ext + entry0 * ext_bs + ((u64)d * ext_limbs + x) * n + jsrc;
                const u64 bs = own ? own_bs : ext_bs;
#pragma unroll
                for (int u = 0; u < IPS_BCH; u++)
                    if (u < live) e[i][u] = src[u * bs];
            }
            if (with_c0) {
#pragma unroll
                for (int u = 0; u < IPS_BCH; u++)
                    if (u < live) c0[u] = ((const double*)c0_src)[(entry0 + u) * own_bs + (u64)x * n + jsrc];
            }
#pragma unroll
            for (int i = 0; i < AT_ONCE; i++) {
#pragma unroll
                for (int u = 0; u < IPS_BCH; u++) {
                    if (u >= live) break;
                    if (d0 + i == own_digit) e[i][u] = fp_norm(fp_from_u64((u64)__double_as_longlong(e[i][u])), p, pinv);
                    fp_sum_add(sb[u], e[i][u], kb[i]);
                    fp_sum_add(sa[u], e[i][u], ka[i]);
                }
            }
            if (with_c0) {
#pragma unroll
                for (int u = 0; u < IPS_BCH; u++)
                    if (u < live) tc[u] += fp_from_u64((u64)__double_as_longlong(c0[u]));
                if (GROUPS == 1 && ++c0_pending == 6) {              // six and a normalised value
                    c0_pending = 0;
#pragma unroll
                    for (int u = 0; u < IPS_BCH; u++) tc[u] = fp_norm(tc[u], p, pinv);
                }
            }
        }
        if (++pending == fold_every) {
            pending = 0;
#pragma unroll
            for (int u = 0; u < IPS_BCH; u++) { fold(sb[u]); fold(sa[u]); }
        }
    }
    static_assert(FP_MAX_STEPS <= 32, "eight rotations a wave of four");
    auto finish = [&](u64 b, double vb, double va, double vc) {
        if (x < l) {
            const double pm = fp_from_u64(pmod[prime]);
            if (plain) {
                const u64* add = plain + b * plain_bs + (u64)x * n + j;
                vc += fp_from_u64(add[0]);
                va += fp_mulmod(fp_from_u64(add[(u64)l * n]), pm, p, pinv);
            }
            vb += fp_mulmod(vc, pm, p, pinv);
        }
        u64* dst = acc + b * acc_bs;
        dst[(u64)x * n + j] = fp_canonical(vb, p, pinv);
        dst[((u64)ext_limbs + x) * n + j] = fp_canonical(va, p, pinv);
    };
#pragma unroll
    for (int u = 0; u < IPS_BCH; u++) { fold(sb[u]); fold(sa[u]); tc[u] = fp_norm(tc[u], p, pinv); }
    if constexpr (GROUPS == 1) {
#pragma unroll
        for (int u = 0; u < IPS_BCH; u++)
            if (u < live) finish(b0 + u, sb[u].l, sa[u].l, tc[u]);
    } else {
        static_assert(GROUPS == IPS_BCH, "a wave finishes an output");
        __shared__ double part[GROUPS][IPS_BCH][3][64];
#pragma unroll
        for (int u = 0; u < IPS_BCH; u++) {
            part[wave][u][0][lane] = sb[u].l;
            part[wave][u][1][lane] = sa[u].l;
            part[wave][u][2][lane] = tc[u];
        }
        __syncthreads();
        if (wave >= live) return;
        double sum[3] = {};
#pragma unroll
        for (int w = 0; w < GROUPS; w++)
#pragma unroll
            for (int i = 0; i < 3; i++) sum[i] += part[w][wave][i][lane];
        finish(b0 + wave, sum[0], sum[1], sum[2]);
    }
}

#define SUM_PARAMS                                                                                                                        \
    const FpPrime *fprimes, const double *ext, u64 ext_bs, int digits, int l, int K, int L, int alpha, IpSteps steps, int n_steps, int total, \
        const u64 *own_src, u64 own_bs, u64 *acc, u64 acc_bs, u64 n_batch, int shared_input, const u64 *c0_src, const u64 *plain,         \
        u64 plain_bs, const u64 *pmod, int log_n
#define SUM_ARGS                                                                                                                   \
    fprimes, ext, ext_bs, digits, l, K, L, alpha, steps, n_steps, total, own_src, own_bs, acc, acc_bs, n_batch, shared_input, c0_src, \
        plain, plain_bs, pmod, log_n
template <int GROUPS, int DIGITS>
__global__ __launch_bounds__(IPF_NT) void inner_product_sum_fp_kernel(SUM_PARAMS) {
    inner_product_sum<GROUPS, DIGITS, false>(SUM_ARGS);
}
template <int GROUPS, int DIGITS>
__global__ __launch_bounds__(IPF_NT) void inner_product_sum_once_kernel(SUM_PARAMS) {
    inner_product_sum<GROUPS, DIGITS, true>(SUM_ARGS);
}

hipError_t launch_inner_product_sum_fp(const FpPrime* fprimes, const double* ext, u64 ext_bs, int digits, int l, int K, int L,
                                       int alpha, const IpSteps& steps, int n_steps, int total, const u64* own_src, u64 own_bs,
                                       u64* acc, u64 acc_bs, u64 n_batch, int shared_input, const u64* c0_src, const u64* plain,
                                       u64 plain_bs, const u64* pmod, int log_n, hipStream_t st) {
    DRY_RUN_RETURN();
    if (digits < 1 || digits > IPF_MAXD || n_steps < 1 || n_steps > FP_MAX_STEPS || l < 1 || K < 1 || alpha < 1) return hipErrorInvalidValue;
    if (!fprimes || !ext || !own_src || !acc || !c0_src || !pmod || n_batch == 0 || n_batch > 65535 || l + K > 65535)
        return hipErrorInvalidValue;
    // an entry holds `digits` extended digits of l + K limbs; an accumulator two polynomials of l + K limbs; an own-digit
    // source and a c0 the l limbs of a polynomial, a plain entry both
    const u64 n = (u64)1 << log_n;
    if (ext_bs < (u64)digits * (l + K) * n || acc_bs < (u64)2 * (l + K) * n || own_bs < (u64)l * n || (plain && plain_bs < (u64)2 * l * n))
        return hipErrorInvalidValue;
    for (int s = 0; s < n_steps; s++)
        if (!steps.key[s] || steps.galois[s] == 0) return hipErrorInvalidValue;
    const unsigned groups_of_outputs = (unsigned)((n_batch + IPS_BCH - 1) / IPS_BCH);
    const bool few = ((u64)groups_of_outputs * (l + K) << log_n) / IPF_NT < IPS_FEW;
    dim3 grid((1u << log_n) / (few ? 64 : IPF_NT), groups_of_outputs, l + K);
    const bool once = groups_of_outputs == 1 && ((u64)n_steps * digits * 2 * (l + K) << (log_n + 3)) > STREAMED_KEY_BYTES;
    ProfScope prof__(once ? "inner_product_sum_once_kernel" : "inner_product_sum_fp_kernel", st);
#define SUM_LAUNCH(G, D)                                                                                                \
    if (once) hipLaunchKernelGGL((inner_product_sum_once_kernel<G, D>), grid, dim3(IPF_NT), 0, st, SUM_ARGS);            \
    else hipLaunchKernelGGL((inner_product_sum_fp_kernel<G, D>), grid, dim3(IPF_NT), 0, st, SUM_ARGS);                   \
    break
    switch ((few ? 4 : 0) + (digits < 4 ? digits : 0)) {
        case 1: SUM_LAUNCH(1, 1);
        case 2: SUM_LAUNCH(1, 2);
        case 3: SUM_LAUNCH(1, 3);
        case 0: SUM_LAUNCH(1, 0);
        case 5: SUM_LAUNCH(4, 1);
        case 6: SUM_LAUNCH(4, 2);
        case 7: SUM_LAUNCH(4, 3);
        default: SUM_LAUNCH(4, 0);
    }
#undef SUM_LAUNCH
#undef SUM_ARGS
#undef SUM_PARAMS
    return hipGetLastError();
}

hipError_t launch_inner_product_steps_fp(const FpPrime* fprimes, const double* ext, u64 ext_bs, int digits, int l, int K, int L,
                                         int alpha, const IpSteps& steps, int n_steps, int total, const u64* own_src,
                                         u64 own_bs, u64* acc, u64 acc_bs, u64 n_batch, int log_n, hipStream_t st,
                                         const u64* c0_src, const u64* pmod) {
    DRY_RUN_RETURN();
    if (digits > IPF_MAXD || n_steps < 1 || n_steps > FP_MAX_STEPS) return hipErrorInvalidValue;
    if (!fprimes || !ext || !own_src || !acc || n_batch == 0 || (c0_src && !pmod)) return hipErrorInvalidValue;
    for (int s = 0; s < n_steps; s++)
        if (!steps.key[s] || steps.galois[s] == 0) return hipErrorInvalidValue;
    dim3 grid((1u << log_n) / IPF_NT, n_steps, l + K);
    ProfScope prof__("inner_product_steps_fp_kernel", st);
    hipLaunchKernelGGL(inner_product_steps_fp_kernel, grid, dim3(IPF_NT), 0, st, fprimes, ext, ext_bs, digits, l, K, L, alpha,
                       steps, total, own_src, own_bs, acc, acc_bs, n_batch, c0_src, pmod, log_n);
    return hipGetLastError();
}
