// The counter-based generator behind every random polynomial, device side: two rounds of a 64-bit mixer, the first over
// seed and stream (kind, counter), the second over the index.
#pragma once
#include <stdint.h>

typedef uint64_t u64;
typedef int64_t i64;

__device__ __forceinline__ u64 mix64(u64 x) {
    x ^= x >> 32; x *= 0x6a09e667f3bcc909ULL;
    x ^= x >> 29; x *= 0xbb67ae8584caa73bULL;
    x ^= x >> 32;
    return x;
}
__device__ __forceinline__ u64 stream_key(u64 seed, u64 kind, u64 ctr) {
    return mix64(seed + 0x3c6ef372fe94f82bULL * (((kind << 56) | ctr) + 1));
}
__device__ __forceinline__ u64 rnd_at(u64 key, u64 idx) { return mix64(key + 0x3c6ef372fe94f82bULL * (idx + 1)); }

// a word of the stream as a sample of the error distribution: the magnitude is the number of entries of the cumulative
// table (floor(2^63 P(|X| <= k)), k < cdt_n) that its upper 63 bits reach, the sign its low bit
__device__ __forceinline__ i64 gaussian_from_word(u64 w, const u64* cdt, int cdt_n) {
    const u64 mag_src = w >> 1;
    i64 mag = 0;
    for (int k = 0; k < cdt_n; k++) mag += (mag_src >= cdt[k]);
    return (w & 1) ? -mag : mag;
}
// the same for R words at once: an entry of the table, which is fetched from memory, serves them all
template <int R>
__device__ __forceinline__ void gaussians_from_words(double (&v)[R], const u64 (&w)[R], const u64* cdt, int cdt_n) {
    int mag[R] = {};
#pragma unroll 4
    for (int k = 0; k < cdt_n; k++) {
        const u64 c = cdt[k];
#pragma unroll
        for (int r = 0; r < R; r++) mag[r] += (w[r] >> 1) >= c;
    }
#pragma unroll
    for (int r = 0; r < R; r++) v[r] = (double)(w[r] & 1 ? -mag[r] : mag[r]);
}
