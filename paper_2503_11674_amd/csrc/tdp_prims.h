// Device primitives shared by the HIP sources (scan, radix sort, fills).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace tdp {
// Exclusive prefix sum of in[0..n) into out (may alias in); n = min(cap, *d_n)
// when d_n is given.  *d_total (optional) receives the sum.  tmp needs
// scan_tmp_size(cap) ints.
void scan_exclusive(const int32_t *in, int32_t *out, int cap, const int32_t *d_n, int32_t *d_total,
                    int32_t *tmp, hipStream_t s);
int scan_tmp_size(int cap);
// Stable sort of the low `bits` bits of 32- or 64-bit keys carrying 32-bit
// values, by digits of at most digit_bits (<= 11) bits; the result is in one of
// the two pairs of buffers.  n = min(cap, *d_n) when d_n is given.  hist needs
// sort_hist_size(cap, digit_bits) ints.
template <typename Key> struct Sorted { Key *keys; uint32_t *vals; };
template <typename Key>
Sorted<Key> radix_sort(Key *k0, uint32_t *v0, Key *k1, uint32_t *v1, int cap, const int32_t *d_n, int bits,
                       int digit_bits, int32_t *hist, hipStream_t s);
int sort_hist_size(int cap, int digit_bits);
void fill_i32(int32_t *p, int n, int32_t v, hipStream_t s);
// xy[i] = (x[i], y[i]): one 8-byte gather per random position lookup; where
// a coordinate is NaN or infinite, *bad = gen (if bad is given); tag (if
// given) notes whether err has bit 1 set and, with a note, counts the arrival
// passes; *note (if given) = noted
void pack_xy(const float *x, const float *y, float2 *xy, int n, hipStream_t s, int32_t *bad = nullptr,
             int32_t gen = 0, const int32_t *err = nullptr, uint32_t *tag = nullptr, uint32_t *note = nullptr,
             uint32_t noted = 0);

// order-preserving maps from floating point to unsigned integers
__host__ __device__ __forceinline__ uint64_t order_key(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (uint64_t)((u & 0x80000000u) ? ~u : (u | 0x80000000u));
}
__host__ __device__ __forceinline__ uint64_t order_key(double f) {
  uint64_t u = __builtin_bit_cast(uint64_t, f);
  return (u & 0x8000000000000000ull) ? ~u : (u | 0x8000000000000000ull);
}
}  // namespace tdp
