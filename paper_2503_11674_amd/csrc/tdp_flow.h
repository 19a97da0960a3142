// Dataflow sweeps' building blocks: words that a wave of a resident grid waits
// for, and the grid's size.
#pragma once

#include <algorithm>

#include "tdp_wave.h"

namespace tdp {

// published words of the dataflow sweeps (relaxed device-scope atomics; a
// consumer polls one word, so no fences are needed)
constexpr uint64_t W_EMPTY = ~0ull;
// a published required time: its bits, all ones = not yet (no computed value,
// NaN included, has that pattern)
template <typename T> struct ReqWord;
template <> struct ReqWord<float> {
  using type = uint32_t;
  static __device__ __forceinline__ uint32_t bits(float v) { return __float_as_uint(v); }
  static __device__ __forceinline__ float value(uint32_t w) { return __uint_as_float(w); }
};
template <> struct ReqWord<double> {
  using type = uint64_t;
  static __device__ __forceinline__ uint64_t bits(double v) { return (uint64_t)__double_as_longlong(v); }
  static __device__ __forceinline__ double value(uint64_t w) { return __longlong_as_double((long long)w); }
};

// Poll *p until it differs from `empty`, with one short sleep between polls
// (a longer back-off delays the frontier by the sleep).  The wait is
// bounded: after `limit` polls (or once another wave has given up) it sets
// bit 2 of *err and returns `empty`, so every wave always finishes.
template <typename U>
__device__ __forceinline__ U wait_pub(const U *p, U empty, int32_t *err, int limit) {
  U v = pub_ld(p);
  int it = 0;
  while (v == empty) {
    if (++it > limit) {
      atomicOr(err, 2);
      break;
    }
    if ((it & 31) == 0 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) break;
    __builtin_amdgcn_s_sleep(1);
    v = pub_ld(p);
  }
  return v;
}

// A wave first waits on one representative word with its lane 0 alone (the
// word its chunk is likely to see published last), so that a waiting wave
// polls one address rather than 64; every lane then checks its own word.
template <typename U>
__device__ __forceinline__ void wait_rep(const U *p, U empty, int32_t *err, int limit) {
  if (wave_lane() == 0) (void)wait_pub(p, empty, err, limit);
}

// Every lane that wants one loads its word; only if some wanted word is not
// yet published does the wave wait: one lane polls the missing word that is
// published last (the highest-numbered one when producers go up the index
// order, the lowest with LOW_LAST), then the missing lanes wait for theirs.
// A wave behind the frontier pays one memory round trip.  Lanes that want
// nothing get `empty`.
template <bool LOW_LAST = false, typename U>
__device__ __forceinline__ U load_or_wait(const U *base, int idx, bool want, U empty, int32_t *err, int limit) {
  U v = want ? pub_ld(base + idx) : empty;
  const bool miss = want && v == empty;
  if (__ballot(miss)) {
    const int rep = LOW_LAST ? -wave_max_int(miss ? -idx : INT32_MIN + 1) : wave_max_int(miss ? idx : -1);
    if (wave_lane() == 0) (void)wait_pub(base + rep, empty, err, limit);
    if (miss) v = wait_pub(base + idx, empty, err, limit);
  }
  return v;
}

// workgroups of `waves` waves of a kernel that a compute unit holds (cached per wave count)
inline int occupancy(const void *kern, int32_t *occ_cache, int waves, size_t lds) {
  const int wi = waves == 1 ? 0 : (waves == 2 ? 1 : 2);
  if (occ_cache[wi] < 0) {
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, 64 * waves, lds) != hipSuccess || occ < 1) occ = 1;
    occ_cache[wi] = occ;
  }
  return occ_cache[wi];
}

// `per` resident workgroups per compute unit, but no more than `units` of work (one per wave) need
inline int resident_blocks(tdp_graph g, int per, int waves, int units) {
  return (int)std::max(1LL, std::min((long long)std::max(1, per) * std::max(1, g->num_cu), (long long)(units + waves - 1) / waves));
}

}  // namespace tdp
