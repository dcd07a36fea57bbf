// Negacyclic NTT / inverse NTT over Z_q[X]/(X^N+1), N = 2^10 .. 2^16, batched over limb-polynomials.  Forward: natural order
// in, a(psi^(2*bitrev(i)+1)) at index i out (decimation in time, psi-twist merged into the twiddles).  Inverse: the same levels
// undone in reverse order, then N^-1.  This file chooses the kernels: exact fp64 (primes below 2^50, N = 2^12 .. 2^15; by
// columns and rows or, for many polynomials, a workgroup each) or 64-bit integers by columns and rows.
#include "hisa_internal.hpp"

// PolyMap -> compact task list of the fp64 single-launch transform; false when it does not fit
static bool fp_tasks(const NttTables& t, int log_n, const PolyMap& map, int n_polys, FpTask* tk) {
    if (!t.fp_ok || log_n < 12 || log_n > 15 || n_polys % map.period != 0) return false;
    int cnt = 0;
    for (int e = 0; e < map.period; e++) {
        if (map.prime_of[e] < 0) continue;
        if (cnt >= HISA_MAX_PRIMES) return false;
        tk->pos[cnt] = (int16_t)e;
        tk->prime[cnt] = map.prime_of[e];
        cnt++;
    }
    tk->period = cnt;
    return cnt > 0;
}

static void int_tasks(const PolyMap& map, IntTasks* tk) {
    tk->n = 0;
    for (int e = 0; e < map.period; e++) {
        if (map.prime_of[e] < 0) continue;
        tk->pos[tk->n] = (int16_t)e;
        tk->prime[tk->n++] = map.prime_of[e];
    }
}

IntArgs int_base_args(const NttTables& t, int log_n) {
    IntArgs a = {};
    a.primes = t.primes; a.tw = t.tw; a.tw_sh = t.tw_sh; a.itw = t.itw; a.itw_sh = t.itw_sh; a.consts = t.consts;
    a.log_n = log_n;
    return a;
}

static FpArgs fp_base_args(const NttTables& t) {
    FpArgs a = {};
    a.fprimes = t.fprimes; a.ftw = t.ftw; a.utw = t.utw; a.vtw = t.vtw; a.sfwd = t.sfwd; a.sinv = t.sinv;
    return a;
}

// By columns and rows up to about the number of polynomials the single-launch transform keeps resident: it takes as long
// for one as for that many.
static bool few_polynomials(int log_n, u64 polys) { return (polys << log_n) <= FEW_COEFFS; }

static hipError_t transform_fp(int mode, int log_n, const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st) {
    return few_polynomials(log_n, n_batch * (u64)tk.period) ? launch_ntt_fp_split(mode, log_n, a, tk, n_batch, st)
                                                            : launch_ntt_fp(mode, log_n, a, tk, n_batch, st);
}

hipError_t launch_ntt_i64(const NttTables& t, int log_n, const i64* coeffs, u64* out, int limbs, int n_pts, hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_pts <= 0) return hipSuccess;
    const PolyMap map = identity_map(limbs);
    FpTask tk;
    if (fp_tasks(t, log_n, map, n_pts * limbs, &tk) && few_polynomials(log_n, (u64)n_pts * limbs)) {
        FpArgs fa = fp_base_args(t);
        fa.coeffs = coeffs; fa.out = out; fa.out_bs = (u64)limbs << log_n;
        return launch_ntt_fp_split(FP_FWD_PLAIN, log_n, fa, tk, (u64)n_pts, st);
    }
    if (!t.fp_ok) {
        IntTasks it;
        int_tasks(map, &it);
        IntArgs a = int_base_args(t, log_n);
        a.n_entries = (unsigned)n_pts;
        a.coeffs = coeffs; a.out = out; a.out_bs = (u64)limbs << log_n;
        return launch_ntt_int(a, it, st);
    }
    hipError_t e = launch_reduce_i64(t.primes, coeffs, out, limbs, n_pts, log_n, st);
    return e == hipSuccess ? launch_ntt(t, log_n, out, (u64)limbs << log_n, n_pts * limbs, map, st) : e;
}

// (in the form for few polynomials: what is decoded comes in groups below that line)
hipError_t launch_intt_centred(const NttTables& t, int log_n, const u64* in, double* out, int limbs, int n_pts, hipStream_t st) {
    DRY_RUN_RETURN();
    FpTask tk;
    if (!fp_tasks(t, log_n, identity_map(limbs), n_pts * limbs, &tk)) return hipErrorInvalidValue;
    FpArgs fa = fp_base_args(t);
    fa.in = in; fa.in_bs = (u64)limbs << log_n; fa.out = (u64*)out; fa.out_bs = (u64)limbs << log_n; fa.centred_out = 1;
    return launch_ntt_fp_split(FP_INV_PLAIN, log_n, fa, tk, (u64)n_pts, st);
}

hipError_t launch_ntt(const NttTables& t, int log_n, u64* data, u64 batch_stride, int n_polys, const PolyMap& map,
                      hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_polys <= 0) return hipSuccess;
    FpTask tk;
    if (fp_tasks(t, log_n, map, n_polys, &tk)) {
        FpArgs fa = fp_base_args(t);
        fa.in = data; fa.in_bs = batch_stride; fa.out = data; fa.out_bs = batch_stride;
        return transform_fp(FP_FWD_PLAIN, log_n, fa, tk, (u64)(n_polys / map.period), st);
    }
    IntTasks it;
    int_tasks(map, &it);
    if (n_polys % map.period) return hipErrorInvalidValue;
    IntArgs a = int_base_args(t, log_n);
    a.n_entries = (unsigned)(n_polys / map.period);
    a.in = data; a.in_bs = batch_stride; a.out = data; a.out_bs = batch_stride;
    return it.n ? launch_ntt_int(a, it, st) : hipSuccess;
}

hipError_t launch_intt(const NttTables& t, int log_n, const u64* in, u64* out, u64 batch_stride, int n_polys, const PolyMap& map,
                       hipStream_t st) {
    DRY_RUN_RETURN();
    if (n_polys <= 0) return hipSuccess;
    FpTask tk;
    if (fp_tasks(t, log_n, map, n_polys, &tk)) {
        FpArgs fa = fp_base_args(t);
        fa.in = in; fa.in_bs = batch_stride; fa.out = out; fa.out_bs = batch_stride;
        return transform_fp(FP_INV_PLAIN, log_n, fa, tk, (u64)(n_polys / map.period), st);
    }
    IntTasks it;
    int_tasks(map, &it);
    if (n_polys % map.period) return hipErrorInvalidValue;
    IntArgs a = int_base_args(t, log_n);
    a.n_entries = (unsigned)(n_polys / map.period);
    a.in = in; a.in_bs = batch_stride; a.out = out; a.out_bs = batch_stride;
    return it.n ? launch_intt_int(a, it, st) : hipSuccess;
}
