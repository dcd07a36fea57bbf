// Internal declarations shared by the translation units of libhisa.
// Host orchestration lives in hisa_api.hip; every arithmetic step runs in the
// kernels declared here (launch wrappers take plain pointers and sizes).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <map>
#include <set>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/hisa.h"

typedef uint64_t u64;
typedef int64_t i64;
typedef unsigned __int128 u128;

// Per-prime constants, one entry per prime q_0..q_{L-1}, p_0..p_{K-1}, device resident.
struct PrimeConst {
    u64 q;
    u64 r1, r0;        // floor(2^128 / q)
    u64 n_inv, n_inv_sh; // N^-1 mod q and its Shoup companion
    u64 half;          // floor(q / 2)
};

// fp64 view of a prime below 2^50 (exact modular arithmetic in doubles)
struct FpPrime {
    double p, pinv, half;
    double ninv;       // N^-1 mod p, centred
};

// Device pointers to the per-prime tables, [prime][N] each.
struct NttTables {
    const PrimeConst* primes;
    const u64* tw;     // psi^bitrev(i)
    const u64* tw_sh;  // Shoup companions
    const u64* itw;    // psi^-bitrev(i)
    const u64* itw_sh;
    const u64* consts; // per prime: N^-1 and N^-1 times itw[1] with companions, floor(2^(63 + bits) / q), bits - 1 (convert_int.hip)
    // fp64 path (all primes below 2^50, 12 <= log2 N <= 15), else fp_ok = 0 and the pointers are null
    int fp_ok;
    const FpPrime* fprimes;
    const double* ftw;  // psi^bitrev(i), centred
    const double* utw;  // utw[m + k] = psi^(-k N/m), k < m = 2^t: inverse decimation-in-time twiddles
    const double* vtw;  // psi^-j / N
    const double *sfwd, *sinv;   // twiddles of the row / column kernels (convert_fp.hip), split_table_words(log_n) per prime
};

// Which polynomials a batched NTT launch touches: polynomial p (0 <= p <
// n_polys) sits at base + (p / period) * batch_stride + (p % period) * N and
// is transformed modulo prime prime_of[p % period]; a negative entry skips it.
#define HISA_MAX_PERIOD 256
struct PolyMap {
    int32_t period;
    int16_t prime_of[HISA_MAX_PERIOD];
};

// One fast base conversion: source primes src[0..a), all primes as targets.
struct ConvTable {
    int a;
    int src[HISA_MAX_Q];
    std::vector<u64> inv_hat; // [a]         (D/c_i)^-1 mod c_i
    std::vector<u64> hat;     // [a][total]  (D/c_i) mod t
    double* d_hat_f;    // [a][total]  (D/c_i) mod t as centred doubles (fp64 path), may be null
};

struct DevBlock {
    void* ptr;
    size_t bytes;
    int refs;
};

#define HISA_MAGIC_CT 0x43544631u
#define HISA_MAGIC_PT 0x50544631u

struct hisa_ct {
    uint32_t magic;
    DevBlock* blk;
    u64* data;  // [polys][limbs][N], NTT form
    uint32_t polys, limbs;
    double scale;
};

struct hisa_pt {
    uint32_t magic;
    DevBlock* blk;
    u64* data;  // [limbs][N], NTT form
    uint32_t limbs;
    double scale;
};

struct SwitchKey {
    DevBlock* blk;
    u64* data;  // [dnum][2][total][N]: b then a, NTT form; centred doubles where the fused path is available, else residues
};

struct hisa_ctx {
    hisa_params prm;
    uint32_t log_n, N, L, K, alpha, dnum, total;
    hipStream_t stream;
    std::vector<u64> mod, psi;  // q_0..q_{L-1}, p_0..p_{K-1}
    std::vector<PrimeConst> pc;
    PrimeConst* d_primes;
    u64 *d_tw, *d_tw_sh, *d_itw, *d_itw_sh;
    NttTables tabs;
    u64* d_secret;  // [total][N], NTT form
    std::map<u64, SwitchKey> keys;  // 0: relinearisation, else Galois element
    struct Analysis* analysis = nullptr;   // non-null between hisa_analysis_begin and hisa_analysis_end
    uint32_t fused_rescale = 0;            // hisa_set_fused_rescale: layers divide by q_{l-1} P at once where they can
    uint32_t merge_doublings = 0;          // hisa_set_merge_doublings: rotate-and-add chains as sums of rotations (0, 2..4)
    std::map<u64, SwitchKey> aux;   // small derived device tables, built on first use
    std::map<std::pair<int, int>, ConvTable> modup_tabs;  // (digit, size)
    ConvTable* moddown_tab;
    std::vector<u64> pinv;       // [L] P^-1 mod q_i
    u64* d_consts;    // NttTables::consts
    std::vector<u64> last_itw;   // inverse twiddle of the level that pairs the two halves, per prime
    u64* d_pmod;      // [L] P mod q_i
    double *d_cos, *d_sin;  // [2N] roots of unity exp(i*pi*t/N)
    FpPrime* d_fprimes;     // fp64 path tables (null when not applicable)
    double *d_ftw, *d_utw, *d_vtw, *d_pinv_f;
    double *d_sfwd = nullptr, *d_sinv = nullptr;   // row and column twiddles
    u64* d_gauss_cdt = nullptr;            // [gauss_cdt_n] floor(2^63 P(|X| <= k)) of the error distribution
    int gauss_cdt_n = 0;
    std::vector<i64> sparse_secret;        // secret_kind = 1: the secret's coefficients, drawn on the host
    double* d_moddown_hat_pin = nullptr;   // [K][total] (P/p_m) * P^-1 mod q_i, centred: ModDown's conversion with the division folded in
    double* d_sfft_tw = nullptr;           // [N/2] complex: stage twiddles of the encode / decode transform
    unsigned char* pin = nullptr;          // pinned host memory that uploads and decoded values pass through (pinned_block)
    size_t pin_pos = 0;
    std::unordered_map<size_t, std::vector<void*>> pool;
    size_t pool_bytes;
    std::map<uintptr_t, size_t> live;   // blocks handed out by dev_alloc and not yet back in the pool: start -> bytes
    u64 enc_counter;
    int device = -1;              // the GPU the context lives on (current when it was made)
    void* noalloc_ws = nullptr;   // that GPU's copy of the library's static scratch array (hisa_rot_left_noalloc)
    std::string err;
};

// ---- host helpers shared by hisa_api.hip and layers.hip ----
int fail(hisa_ctx* ctx, int code, const char* fmt, ...);

#define HIP_TRY(ctx, expr)                                                                        \
    do {                                                                                          \
        hipError_t e__ = (expr);                                                                  \
        if (e__ != hipSuccess)                                                                    \
            return fail(ctx, e__ == hipErrorOutOfMemory ? HISA_ERR_OOM : HISA_ERR_HIP, "%s: %s", #expr, \
                        hipGetErrorString(e__));                                                  \
    } while (0)

#define TRY(expr)                  \
    do {                           \
        int rc__ = (expr);         \
        if (rc__ != HISA_OK) return rc__; \
    } while (0)

DevBlock* dev_alloc(hisa_ctx* ctx, size_t bytes);   // from the context's pool; null (and last_error set) on failure
void dev_release(hisa_ctx* ctx, DevBlock* b);
// 8-byte words from p to the end of the live pool block that holds p; 0 when no live block does
u64 dev_words_behind(const hisa_ctx* ctx, const void* p);

// `bytes` (at most PIN_BYTES) of pinned host memory, readable and writable by kernels.  The host may use it until the next
// call of this function, kernels enqueued before that call for as long as they run: the memory is a ring, and before it starts
// over the stream is waited for.  A caller that needs two blocks at a time asks for one of twice the size.
#define PIN_BYTES ((size_t)4 << 20)
int pinned_block(hisa_ctx* ctx, size_t bytes, double** out);
// slot values in pinned memory, [n_pts][count] -> plaintexts out [n_pts][limbs][N]; im may be null
int encode_dense(hisa_ctx* ctx, const double* re, const double* im, int count, int n_pts, double scale, int limbs, u64* out);
// plaintexts [n_pts][limbs][N] (device) -> the first `count` slots, complex z [n_pts][count] in pinned memory; waits
// (n_pts: at most what client_group allows)
int decode_dense(hisa_ctx* ctx, const u64* pts, int n_pts, int limbs, double scale, int count, double* z);

// Coefficients of a set of transforms up to which the two launches over columns and rows are used (ntt.hip)
#define FEW_COEFFS ((u64)1 << 22)
// Plaintexts of `limbs` limbs that one set of encode or decode launches takes: FEW_COEFFS coefficients (4096 rows, which
// fill the chip) bound its scratch to under 100 MB whatever the tensor, and, with N >= 2^10, its grids to 4096 rows of entries.
inline size_t client_group(const hisa_ctx* ctx, size_t limbs) {
    const size_t most = (size_t)FEW_COEFFS / (limbs * ctx->N);
    return most ? most : 1;
}

struct Temp {  // pooled scratch buffer for the duration of one call
    hisa_ctx* ctx;
    DevBlock* blk;
    struct None {};    // no buffer: the caller brought memory of its own
    Temp(hisa_ctx* c, size_t bytes) : ctx(c), blk(dev_alloc(c, bytes)) {}
    Temp(hisa_ctx* c, None) : ctx(c), blk(nullptr) {}
    Temp(hisa_ctx* c, size_t bytes, bool wanted) : ctx(c), blk(wanted ? dev_alloc(c, bytes) : nullptr) {}
    ~Temp() { dev_release(ctx, blk); }
    bool ok() const { return blk != nullptr; }
    u64* u() const { return (u64*)blk->ptr; }
    template <class T> T* as() const { return (T*)blk->ptr; }
    Temp(const Temp&) = delete;
    Temp& operator=(const Temp&) = delete;
};

static inline bool valid_ct(const hisa_ct* c) { return c && c->magic == HISA_MAGIC_CT; }
static inline bool valid_pt(const hisa_pt* p) { return p && p->magic == HISA_MAGIC_PT; }
static inline size_t ct_words(const hisa_ctx* ctx, uint32_t polys, uint32_t limbs) { return (size_t)polys * limbs * ctx->N; }

// n ciphertext handles that are views of one allocation, [n][polys][limbs][N]
int alloc_ct_batch(hisa_ctx* ctx, size_t n, uint32_t polys, uint32_t limbs, double scale, hisa_ct** out);
int alloc_pt(hisa_ctx* ctx, uint32_t limbs, double scale, hisa_pt** out);

// A batch of equally shaped ciphertexts as one strided array.  When the handles are not evenly
// spaced views of one allocation they are first copied side by side (tmp then owns the copy).
struct BatchIn {
    const u64* base = nullptr;
    u64 stride = 0;
    DevBlock* tmp = nullptr;
};
int gather_batch(hisa_ctx* ctx, const hisa_ct* const* cts, size_t n, BatchIn* bi);
int check_batch_shape(hisa_ctx* ctx, const hisa_ct* const* cts, size_t n, uint32_t polys);
PolyMap identity_map(int limbs);
// pieces of the fused fp64 key switch for sums that are formed before the division by P (hisa_api.hip)
bool fused_key_switch_available(const hisa_ctx* ctx);
int rotation_accumulators_fp(hisa_ctx* ctx, const u64* cts, u64 ct_bs, size_t B, int l, const int32_t* steps, int n_steps,
                             u64* acc, bool fold_c0 = false);
// out[b] = plain[b] + sum_s rotLeft(rot[s * Bn + b], steps[s]) with one division by P per output: rot holds
// n_steps * Bn ciphertexts [2][l][N], ct_bs words apart, rotation-major; every step rotates (its key is present);
// plain ([Bn] ciphertexts, plain_bs apart) may be null; out [Bn][2][l][N].  shared_input: rot holds Bn ciphertexts and
// every term of output b rotates rot[b] (one decomposition per output).  Dry runs count and return.
// rescale: the sum's divScalar is taken together with its division by P (moddown_rescale_fp): out [Bn][2][l - 1][N].
int rotate_sum_fp(hisa_ctx* ctx, const u64* rot, u64 ct_bs, int n_steps, const int32_t* steps, size_t Bn, int l,
                  const u64* plain, u64 plain_bs, u64* out, bool shared_input = false, bool rescale = false);
// What a kernel that forms the accumulators of rotations itself reads: the extended digits of B ciphertexts, transformed (ext), the
// keys and automorphisms of the rotations (st)
struct IpSteps;
size_t rotation_digits_bytes(const hisa_ctx* ctx, size_t B, int l);
int rotation_digits_fp(hisa_ctx* ctx, const u64* cts, u64 ct_bs, size_t B, int l, const int32_t* steps, int n_steps, IpSteps* st, double* ext);
// The division by P and the divScalar by q_{l-1} in one base conversion: acc [B][2][l + K][N] (overwritten: the addend
// [B][add_polys][l][N] is first folded in, times P) -> out [B][2][l - 1][N] = (acc + P add) / (q_{l-1} P), rounded as a
// centred conversion rounds.  l >= 2.
int moddown_rescale_fp(hisa_ctx* ctx, u64* acc, size_t B, int l, const u64* add, u64 add_bs, int add_polys, u64* out);
// Relinearisation of n three-polynomial ciphertexts ([3][l][N], stride words apart) whose division by P is taken
// together with the divScalar by q_{l-1}: out [n][2][l - 1][N] = ((d0, d1) + KS_relin(d2)) / q_{l-1}.
int relinearize_rescale_fp(hisa_ctx* ctx, const u64* cts3, u64 stride, size_t n, int l, u64* out);
int moddown_add_fp(hisa_ctx* ctx, const u64* acc, size_t B, int l, const u64* add, u64 add_bs, int add_polys, u64* out);
// exact integer nearest to the double v (ties away from zero), reduced modulo q
u64 double_to_residue(double v, u64 q);

// Optional per-kernel timing with HIP events on the launch stream (off by default; the benchmark
// turns it on for a separate pass).  One scope brackets one kernel launch.
void prof_begin(const char* kernel, hipStream_t st);
void prof_end(hipStream_t st);
extern bool g_prof_on;

// Analysis backend (Sec. "Compiler": the analyser runs the circuit on a HISA backend that records instead of
// computing).  While a context is in analysis mode every launch wrapper returns at once (no kernel runs; memory is
// still allocated, so handles, levels and scales evolve as in a real run) and the primitives count themselves here.
struct Analysis {
    hisa_op_counts c = {};
    std::set<int32_t> steps;    // left-rotation amounts that needed a key
};
extern thread_local Analysis* t_analysis;   // non-null while the calling thread's context is in analysis mode
// n occurrences of an operation on ciphertexts of `limbs` limbs (call only where t_analysis is set)
#define TALLY(field, OP, n, limbs)                                                   \
    do {                                                                             \
        t_analysis->c.field += (uint64_t)(n);                                        \
        t_analysis->c.limb_sum[OP] += (uint64_t)(n) * (uint64_t)(limbs);             \
        t_analysis->c.limb_sq_sum[OP] += (uint64_t)(n) * (uint64_t)(limbs) * (uint64_t)(limbs); \
    } while (0)
#define DRY_RUN_RETURN() do { if (t_analysis) return hipSuccess; } while (0)
struct ProfScope {
    hipStream_t st;
    bool on;
    ProfScope(const char* kernel, hipStream_t s) : st(s), on(g_prof_on) { if (on) prof_begin(kernel, s); }
    ~ProfScope() { if (on) prof_end(st); }
};

// ---- launch wrappers (every one enqueues on `st` and returns hipGetLastError) ----
hipError_t launch_ntt(const NttTables& t, int log_n, u64* data, u64 batch_stride, int n_polys, const PolyMap& map,
                      hipStream_t st);
// signed coefficients [n_pts][N] -> their residues modulo primes 0 .. limbs - 1 in NTT form, out [n_pts][limbs][N]
hipError_t launch_ntt_i64(const NttTables& t, int log_n, const i64* coeffs, u64* out, int limbs, int n_pts, hipStream_t st);
// NTT form [n_pts][limbs][N] -> coefficients as centred doubles (fp64 contexts only)
hipError_t launch_intt_centred(const NttTables& t, int log_n, const u64* in, double* out, int limbs, int n_pts, hipStream_t st);
// `in` and `out` have the same layout and may be the same
hipError_t launch_intt(const NttTables& t, int log_n, const u64* in, u64* out, u64 batch_stride, int n_polys, const PolyMap& map,
                       hipStream_t st);

// ---- fp64 transforms (primes below 2^50, N = 2^12 .. 2^15) ----
// The stages a launch can belong to: 0 and 1 are the whole-polynomial transforms of ntt_fp.hip, the others the row and
// column kernels of convert_fp.hip.
enum FpMode {
    FP_FWD_PLAIN = 0,      // u64 coefficients in, u64 NTT form out
    FP_INV_PLAIN = 1,      // u64 NTT form in, u64 coefficients out
    FP_INV_TO_Y = 2,       // rows: inverse levels of the source limbs of a conversion
    FP_FWD_CONV = 3,       // columns, rows: conversion of the digits and forward levels -> extended digits (doubles)
    FP_FWD_CONV_FINAL = 4, // columns, rows: the same for a division: out = (acc - transform) * P^-1 (+ addend), canonical
    FP_INV_D_TO_Y = 5,     // rows: forward levels of the digits, key inner product, inverse levels of the division's sources
    FP_FWD_CONV_SUB = 6,   // columns: the division's conversion; rows: key inner product minus the division's transform
    FP_FWD_SUB = 7,        // rows: stored accumulators minus the division's transform (small calls)
};

struct FpTask {
    int32_t period;                      // tasks per batch entry
    int16_t pos[HISA_MAX_PRIMES];        // limb position of the task's polynomial inside a batch entry
    int16_t prime[HISA_MAX_PRIMES];      // its prime
};

#define FP_MAX_DIGITS 8   // digits whose conversions one launch can hold
#define FP_MAX_STEPS 32   // rotations per launch of the shared-decomposition path
struct FpArgs {
    const FpPrime* fprimes;
    const double* ftw;
    const double* utw;
    const double* vtw;
    int n_tasks;                       // filled in by the launcher
    const u64* in; u64 in_bs;          // input [batch][..][N]
    u64* out; u64 out_bs;
    // by columns and rows (launch_ntt_fp_split)
    const double *sfwd, *sinv;
    u64 table_stride;                  // filled in by the launcher, like n_entries
    int n_entries;
    const i64* coeffs;                 // forward: signed coefficients [batch][N] for all limbs of an entry, instead of `in`
    int centred_out;                   // inverse: coefficients as centred doubles instead of residues
};
hipError_t launch_ntt_fp(int mode, int log_n, const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st);
hipError_t launch_ntt_fp_split(int mode, int log_n, const FpArgs& a, const FpTask& tk, u64 n_batch, hipStream_t st);

// symmetric encryption of up to ENCRYPT_MAX plaintexts pt[b] ([limbs][N], NTT form): ct [n_entries][2][limbs][N]
#define ENCRYPT_MAX 64
struct EncryptArgs {
    const FpPrime* fprimes;
    const PrimeConst* primes;
    const double* sfwd;
    u64 table_stride;                  // filled in by the launcher
    const u64* secret;
    u64* ct;
    int limbs, n_entries, noise_on;
    u64 seed, ctr;                     // entry b uses the streams ctr + b
    const u64* cdt;
    int cdt_n;
    const u64* pt[ENCRYPT_MAX];
};
hipError_t launch_encrypt_fp(int log_n, const EncryptArgs& a, hipStream_t st);

// ---- inverse transform -> base conversion -> forward transform by rows and columns (convert_fp.hip) ----
#define SPLIT_ROW 672                        // table words per row of 1024 coefficients
size_t split_table_words(int log_n);         // table words per prime
// Entries [b]; limb position x of an entry belongs to prime x for x < l, L + x - l above.  Sources: limbs
// src_pos0 .. src_pos0 + n_src - 1 of `in`; digit d converts sources src0 .. src0 + a - 1 to every limb 0 .. ext_limbs - 1
// outside [own_lo, own_lo + own_n) and leaves limb x at position out_pos0 + x of the output entry.
struct ConvertArgs {
    const FpPrime* fprimes;
    const double *sfwd, *sinv;
    u64 table_stride;
    int log_n, l, L, total;
    unsigned n_entries;
    const u64* in; u64 in_bs;            // NTT form
    u64 galois;                          // `in` is read through sigma_g (0 = none)
    int src_pos0, n_src;
    const double* post;                  // [n_src] (D/c_i)^-1 of the source's digit, or null: the input carries it
    double* mid;                         // workspace [n_entries][n_src][N]
    int n_digits;
    struct Digit { const double* hat; int src0, a, own_lo, own_n, out_pos0; } dg[8];   // hat: [a][total] (D/c_i) mod t
    int ext_limbs;
    u64* out; u64 out_bs;
    int chunk, n_splits;                 // filled in by the launcher
    // FP_FWD_CONV_FINAL (residues) and FP_FWD_SUB (doubles, |acc| <= 2.75 p): accumulators, limbs in place
    const u64* acc; u64 acc_bs;
    const double* pinv_tab;              // [prime] P^-1 mod q, centred
    // FP_FWD_CONV_FINAL: addend of entry b: add + (b / add_div) * add_bs + (b % add_div) * add_ps, if b % add_div < add_polys
    const u64* add; u64 add_bs, add_ps; int add_div, add_polys;
};
hipError_t launch_inverse_rows_fp(const ConvertArgs& a, hipStream_t st);              // in -> mid
hipError_t launch_columns_fp(int mode, const ConvertArgs& a, hipStream_t st);         // mid -> out (modes 3, 4, 6)
hipError_t launch_forward_rows_fp(int mode, const ConvertArgs& a, hipStream_t st);    // out, in place (modes 3, 4, 7)
// The rows behind the columns of a key switch's digits (ConvertArgs::out: [n_entries][digits][ext_limbs][N]), with the inner
// product with `key` and the neighbouring halves of the division that follows, for the limbs x_begin .. x_end - 1.
// FP_INV_D_TO_Y: limbs from n_acc on are sources of that division: down [n_entries * 2][ext_limbs - n_acc][N] =
// (sum * c1[x] (+ addend * c2[x])) after the inverse rows, `mid` of the division's columns; limbs below n_acc leave as
// acc [n_entries][2][n_acc][N] = sum * c1[x] (+ addend * c2[x]), lazily reduced doubles for FP_FWD_SUB.
// FP_FWD_CONV_SUB (limbs below n_acc): out holds the division's columns and receives its result.
// Own digits and addend are read through sigma_g.
// With StepArgs: several rotations of the same step_B ciphertexts, entry b being rotation b / step_B of ciphertext b % step_B.
// ConvertArgs::out, own and add then hold step_B entries, out fully transformed, normalised digits, and all three are read through
// the rotation's Galois element (key and galois of InnerArgs are not used); sums and results are rotation-major.
struct IpSteps {
    const u64* key[FP_MAX_STEPS];
    uint32_t galois[FP_MAX_STEPS];
};
struct InnerArgs {
    const u64* key;
    const u64* own; u64 own_bs;
    u64 galois;
    int n_acc, x_begin, x_end;
    int split;                           // set by the launcher: a workgroup a polynomial
    const double* c1;                    // [ext_limbs]
    const double* c2;                    // factors of the addend, limbs of q; null: one
    const u64* add; u64 add_bs, add_ps; int add_polys;
    double* acc;
    u64* out;
    double* down;
};
struct StepArgs {
    unsigned step_B;
    IpSteps steps;
};
hipError_t launch_inner_rows_fp(int mode, const ConvertArgs& a, const InnerArgs& g, const StepArgs* steps, hipStream_t st);

// ---- the same division of work in 64-bit integers (convert_int.hip): any ring degree, primes up to 60 bits, any number of
// digits.  Digit d converts sources d * alpha .. (at most n_src) to every limb 0 .. ext_limbs - 1 (with `own`: outside its
// own) and leaves limb x at position d * ext_limbs + x of the output entry.
enum IntMode { INT_INVERSE, INT_FORWARD, INT_CONVERT, INT_INNER };
struct IntTasks {
    int32_t n;                           // polynomials per batch entry
    int16_t pos[HISA_MAX_PERIOD];        // limb position on the output side
    int16_t prime[HISA_MAX_PERIOD];
};
struct IntArgs {
    const PrimeConst* primes;
    const u64 *tw, *tw_sh, *itw, *itw_sh, *consts;
    int log_n, l, L, total;
    unsigned n_entries;
    const u64* in; u64 in_bs;            // NTT form
    int in_pos_shift;                    // input polynomial of task i at pos[i] + in_pos_shift
    u64 galois;                          // `in` is read through sigma_g (0 = none)
    const i64* coeffs;                   // forward transforms: signed coefficients [entry][N] instead of `in`
    u64* out; u64 out_bs;
    int whole;                           // set by the launcher
    int split;                           // set by the launcher: a workgroup a polynomial
    u64* mid;                            // conversions: workspace [n_entries][n_src][N]
    int src_pos0, n_src, alpha, n_digits, own, ext_limbs;
    const u64* close;                    // [n_src] factor of the source, the same times the last inverse twiddle, with companions
    const u64* hat;                      // [n_src][total] (D / c_i) mod t in 30-bit halves
    const u64* off;                      // [n_digits][total] -sum_i floor(c_i / 2) (D / c_i) mod t
    int chunk, n_splits;                 // set by the launcher
    // division rows: out = (acc - transform) * factor[limb] (+ addend of entry b: add + (b / add_div) * add_bs +
    // (b % add_div) * add_ps, if b % add_div < add_polys, through sigma of add_galois); acc below 8 q
    const u64* acc; u64 acc_bs;
    const u64 *factor, *factor_sh;
    const u64* add; u64 add_bs, add_ps; int add_div, add_polys;
    u64 add_galois;
    // inner product rows: ext [n_entries][n_digits][ext_limbs][N] behind the columns, own digits from `in`;
    // sums [n_entries][2][l][N] (below 8 q), down [n_entries][2][ext_limbs - l][N] (behind the inverse rows)
    const u64* ext; u64 ext_bs;
    const u64* key;
    u64 *sums, *down;
};
hipError_t launch_ntt_int(const IntArgs& a, const IntTasks& tk, hipStream_t st);
hipError_t launch_intt_int(const IntArgs& a, const IntTasks& tk, hipStream_t st);
hipError_t launch_inverse_rows_int(const IntArgs& a, hipStream_t st);   // in -> mid
hipError_t launch_columns_int(const IntArgs& a, hipStream_t st);        // mid -> out
hipError_t launch_inner_rows_int(const IntArgs& a, hipStream_t st);     // ext, in -> sums, down
hipError_t launch_divide_rows_int(const IntArgs& a, hipStream_t st);    // out, in place
IntArgs int_base_args(const NttTables& t, int log_n);
// switching keys of the fused path are kept as centred doubles: [n_rows][total][N] in place; back to canonical residues
hipError_t launch_key_to_doubles(const FpPrime* fprimes, u64* key, int n_rows, int total, int log_n, hipStream_t st);
hipError_t launch_key_to_residues(const FpPrime* fprimes, const u64* key, u64* out, int n_rows, int total, int log_n, hipStream_t st);

// acc[s][b][p][x] = sum_j e_j[x] * key_s[j][p][prime(x)] in fp64; e_j[x] comes from ext unless x lies in digit j, then
// from own_src (the NTT-form input itself)
// For n_steps rotations of the same n_batch ciphertexts (extended digits computed once from the unrotated
// polynomial): rotation s uses keys[s] and gathers through galois[s]; acc entries are ordered rotation-major.
// c0_src (with pmod[i] = P mod q_i): the b accumulator also takes P * sigma_s(c0) on the limbs of q, c0 read at
// c0_src + b * own_bs like the own-digit limbs.
hipError_t launch_inner_product_steps_fp(const FpPrime* fprimes, const double* ext, u64 ext_bs, int digits, int l, int K, int L,
                                         int alpha, const IpSteps& steps, int n_steps, int total, const u64* own_src,
                                         u64 own_bs, u64* acc, u64 acc_bs, u64 n_batch, int log_n, hipStream_t st,
                                         const u64* c0_src = nullptr, const u64* pmod = nullptr);

// The sum over n_steps rotations of different ciphertexts: ext / own_src entry s * n_batch + b is term s of output b
// (digits from the unrotated polynomial); acc[b] = sum_s sum_j sigma_s(e_j) * key_s[j] on the l + K limbs.  On the limbs of q
// the accumulators also take P (pmod[i] = P mod q_i) times sum_s sigma_s(c0) (c0_src, entries as own_src) and times the
// polynomials of plain[b] (null: none).  shared_input: every term of output b is entry b.
hipError_t launch_inner_product_sum_fp(const FpPrime* fprimes, const double* ext, u64 ext_bs, int digits, int l, int K, int L,
                                       int alpha, const IpSteps& steps, int n_steps, int total, const u64* own_src, u64 own_bs,
                                       u64* acc, u64 acc_bs, u64 n_batch, int shared_input, const u64* c0_src, const u64* plain,
                                       u64 plain_bs, const u64* pmod, int log_n, hipStream_t st);

// sampling (counter-based generator, both sides of the parity tests implement it)
hipError_t launch_sample_uniform(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr, const PolyMap& map, int n_polys,
                                 u64 batch_stride, u64 ctr_step, u64* out, int log_n, hipStream_t st);
hipError_t launch_sample_small(const PrimeConst* primes, u64 seed, u64 kind, u64 ctr, int noise_on, int ternary,
                               const u64* cdt, int cdt_n, const PolyMap& map, int n_polys, u64 batch_stride, u64 ctr_step,
                               u64* out, i64* raw, int log_n, hipStream_t st);

// element-wise kernels over [batch][polys][limbs][N]
enum ElemOp { OP_ADD = 0, OP_SUB = 1 };
hipError_t launch_addsub(const PrimeConst* primes, const u64* a, const u64* b, u64* out, int op, int limbs, int polys_a,
                         int polys_b, u64 n_batch, u64 a_bs, u64 b_bs, u64 o_bs, int log_n, hipStream_t st);
hipError_t launch_add_const(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int op, int limbs,
                            int polys, int log_n, hipStream_t st);
// entry b is multiplied by plaintext b % pt_period of the pt_period plaintexts at pt
hipError_t launch_mul_plain(const PrimeConst* primes, const u64* a, const u64* pt, u64* out, int limbs, int polys,
                            u64 n_batch, u64 a_bs, u64 o_bs, int log_n, hipStream_t st, unsigned pt_period = 1);
hipError_t launch_mul_const(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int limbs, int polys,
                            int log_n, hipStream_t st);
hipError_t launch_mul_no_relin(const PrimeConst* primes, const u64* a, const u64* b, u64* out, int limbs, u64 n_batch,
                               u64 a_bs, u64 b_bs, u64 o_bs, int log_n, hipStream_t st);
// x^2 + c x of two-polynomial entries as three-polynomial ones; consts: [limbs] residues of c, null: none
hipError_t launch_square_linear(const PrimeConst* primes, const u64* a, u64* out, const u64* consts, int limbs, u64 n_batch, u64 a_bs,
                                u64 o_bs, int log_n, hipStream_t st);
hipError_t launch_encrypt_combine(const PrimeConst* primes, const u64* secret, const u64* pt, const u64* e, u64* ct,
                                  int limbs, u64 n_batch, u64 pt_bs, int log_n, hipStream_t st);
// n_batch ciphertexts ct_bs words apart -> pt [n_batch][limbs][N]
hipError_t launch_decrypt(const PrimeConst* primes, const u64* secret, const u64* ct, u64 ct_bs, u64* pt, int limbs, int polys,
                          u64 n_batch, int log_n, hipStream_t st);
hipError_t launch_key_combine(const PrimeConst* primes, const u64* secret, const u64* target, const u64* e,
                              const u64* pmod_all, u64* key_digit, int total, int L, int alpha, int digit, int log_n,
                              hipStream_t st);
hipError_t launch_pointwise_square(const PrimeConst* primes, const u64* s, u64* out, int total, int log_n, hipStream_t st);
hipError_t launch_automorph_ntt(const u64* in, u64 in_bs, u64* out, u64 out_bs, u64 galois, int n_polys, u64 n_batch,
                                int log_n, hipStream_t st);
#define GALOIS_TAB_MAX 256
struct GaloisTab { uint32_t g[GALOIS_TAB_MAX]; };
// several automorphisms of the same inputs: out entry (s, b) = sigma_{tab.g[s]}(in entry b), entries out_bs words apart
hipError_t launch_automorph_steps(const u64* in, u64 in_bs, u64* out, u64 out_bs, const GaloisTab& tab, int n_steps,
                                  int n_polys, u64 n_batch, int log_n, hipStream_t st);
// acc entries (ciphertext, polynomial), acc_bs apart: acc += P * add on the first l limbs, for polynomials < add_polys
hipError_t launch_fold_addend(const PrimeConst* primes, u64* acc, u64 acc_bs, const u64* add, u64 add_bs, u64 add_ps,
                              int add_polys, const u64* pmod, u64 n_cts, int l, int log_n, hipStream_t st);
hipError_t launch_reduce_i64(const PrimeConst* primes, const i64* coeffs, u64* out, int limbs, int n_pts, int log_n,
                             hipStream_t st);
// the same with the output entries out_limbs limbs apart (residues on a second list of primes go behind the first)
hipError_t launch_reduce_i64(const PrimeConst* primes, const i64* coeffs, u64* out, int limbs, int out_limbs, int n_pts,
                             int log_n, hipStream_t st);

// encode / decode
hipError_t launch_encode(const double* cs, const uint32_t* g, const double* re, int count, int n_pts, double factor, i64* coeffs,
                         int log_n, hipStream_t st);
// piecewise-constant plaintexts: indicator encodings of nb slot sets (g[set_begin[b] .. set_begin[b+1]) lists 5^slot
// mod 2N of set b), then coeffs[p] = round(factor * sum_b v[p][b] * basis[b])
hipError_t launch_encode_basis(const double* cs, const uint32_t* g, const int* set_begin, int nb, double* basis, int log_n,
                               hipStream_t st);
hipError_t launch_encode_combine(const double* basis, int nb, const double* v, int n_pts, double factor, i64* coeffs,
                                 int log_n, hipStream_t st);
// the same maps through the O(N log N) transform over the slot order (encode.hip); tw: [N/2] complex, entry half + j the
// twiddle j of the stage of length 2 half; slot values and z may lie in pinned host memory
hipError_t launch_decode_fft(const void* tw, const double* m, int count, int n_pts, void* work, void* z, int log_n, hipStream_t st);
hipError_t launch_encode_fft(const void* tw, const double* re, const double* im, const uint32_t* slots, int count, int n_pts,
                             double factor, void* work, i64* coeffs, int log_n, hipStream_t st, bool mirror = false);
hipError_t launch_crt_to_double(const PrimeConst* primes, const u64* coeff_form, int limbs, const u64* garner_inv,
                                const u64* garner_inv_sh, int L, double inv_scale, double* out, int n_pts, int log_n, hipStream_t st);
hipError_t launch_crt_fp(const FpPrime* fprimes, const double* centred, int limbs, const double* garner_inv, int L, double inv_scale,
                         double* out, int n_pts, int log_n, hipStream_t st);
hipError_t launch_decode(const double* cs, const double* sn, const double* m, int count, int n_pts, void* z, int log_n, hipStream_t st);
