// Dataflow sweeps' building blocks: words that a wave of a resident grid waits
// for, and the grid's size.
#pragma once

#include <algorithm>

#include "tdp_wave.h"

namespace tdp {

// published words of the dataflow sweeps (relaxed device-scope atomics; a
// consumer polls one word, so no fences are needed)
constexpr uint64_t W_EMPTY = ~0ull;
// a published required time or sum: its bits, all ones = not yet
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

// a value as its word (a NaN may have come in with the positions and have any pattern)
template <typename T>
__device__ __forceinline__ typename ReqWord<T>::type pub_bits(T v) {
  return ReqWord<T>::bits(v == v ? v : (T)__builtin_nan(""));
}

// Shares and tickets.  A resident sweep gives every wave a fixed share of its chunks, which needs all
// its workgroups on the GPU.  Other streams may keep some of them out for as long
// as the ones inside wait: three sweeps of different graphs are more than the GPU
// holds, and each may be dispatched in part.  So a wave that has waited for long
// and finds workgroups that have not begun stops the fixed shares: every wave
// leaves its own where it waits, and the workgroups inside take the chunks from
// the first one on by tickets, computing those already done once more (the same
// values).  The lowest chunk not yet done then has a running owner whichever
// workgroups are inside, so any number of sweeps may run at once.

// What a wait needs besides its word: all but the budget is loaded where it is
// used (by scalar loads), as are the arrays of the code that takes tickets.  As
// kernel arguments they would be held in scalar registers through the loops that
// hardly ever lead there, which then spill.
template <Sweep S>
struct Waits {
  const SweepArgs *device_args;
  int limit;  // polls
  __device__ __forceinline__ const SweepArgs &args() const {
    return *(const SweepArgs *)(const __attribute__((address_space(4))) SweepArgs *)(uintptr_t)device_args;
  }
  __device__ __forceinline__ SweepShare *share() const { return args().share + S; }
  __device__ __forceinline__ int32_t *err() const { return args().err + (S >= SWEEP_ST_FORWARD ? ST_ERR : 0); }
  // [here_stride] the sweep that a workgroup last began
  __device__ __forceinline__ uint32_t *here() const { return args().here + S * args().here_stride; }
};

// polls (some 0.6 us each) before a wave looks for workgroups that have not
// begun: longer than most sweeps take, and than the tail of another stream's
// kernel that a workgroup has to wait for
constexpr int PATIENCE = 512;

// every workgroup, before its first wait
template <Sweep S>
__device__ __forceinline__ void begin_share(const Waits<S> &w) {
  if (threadIdx.x == 0) pub_st(w.here() + blockIdx.x, w.share()->number);
}
// a new sweep, by one thread of the launch that resets the words it publishes
__device__ __forceinline__ void new_sweep(SweepShare *sh) {
  sh->ticket[0] = sh->ticket[1] = 0;
  sh->ended = 0;
  ++sh->number;
}

__device__ __forceinline__ int take_ticket(uint32_t *ticket) {
  int got = 0;
  if (wave_lane() == 0) got = (int)atomicAdd(ticket, 1u);
  return __builtin_amdgcn_readfirstlane(got);
}

// A wave's wait for its words, every lane in it:
//   do {
//     do load; while (polls.missing(some word is not there));
//   } while (polls.resume(the same));
// The inner loop is a part of every level's time and holds no more than it needs
// (with the outer one's steps in it the forward sweep of 200k cells took 221 us,
// not 150): it ends once all lanes have their words, when another wave has ended
// the sweep's waits, or after a run of polls.  A wait is bounded: after `limit`
// polls the wave gives up, sets bit 2 of *err and goes on with what it has, and so
// do all others, so every wave always finishes.  TICKETS: the wave's chunk comes
// from a ticket, and it does not leave.
template <bool TICKETS, Sweep S>
struct Polls {
  const Waits<S> &w;
  int it = 0, run;
  bool leave = false;  // the wave is to leave its fixed share
  __device__ __forceinline__ explicit Polls(const Waits<S> &w) : w(w), run(first_run(w.limit)) {}
  static __device__ __forceinline__ int first_run(int limit) { return TICKETS ? limit : min(PATIENCE, limit >> 4); }
  __device__ __forceinline__ bool missing(bool miss, bool sleep = true) {
    if (!__ballot(miss)) return false;
    if (++it > run) return false;
    if ((it & 31) == 0 && __ballot(pub_ld(&w.share()->ended) != 0)) return false;
    if (sleep) __builtin_amdgcn_s_sleep(1);  // (a longer back-off delays the frontier by the sleep)
    return true;
  }
  __device__ __forceinline__ bool resume(bool miss) {
    if (!__ballot(miss)) return false;
    SweepShare *const sh = w.share();
    const uint32_t ended = pub_ld(&sh->ended);
    if (__ballot((ended & SWEEP_GAVE_UP) != 0)) return false;
    if constexpr (!TICKETS) {
      // the last workgroups to be dispatched, a lane each
      const int b = (int)gridDim.x - 1 - wave_lane();
      const bool out = it > w.limit >> 4 || (b >= 0 && pub_ld(w.here() + b) != sh->number);
      if (__ballot(out) && wave_lane() == 0) atomicOr(&sh->ended, SWEEP_BY_TICKETS);
      leave = __ballot(out || (ended & SWEEP_BY_TICKETS) != 0) != 0;
      if (leave) return false;
      run = min(it + PATIENCE, w.limit >> 4);
      return true;
    }
    if (it <= w.limit) return true;
    if (wave_lane() == 0) {
      atomicOr(w.err(), 2);
      atomicOr(&sh->ended, SWEEP_GAVE_UP);
    }
    return false;
  }
};

// Every lane that wants one loads its word; only if some wanted word is not
// yet published does the wave wait: one lane polls the missing word that is
// published last (the highest-numbered one when producers go up the index
// order, the lowest with LOW_LAST), so that a waiting wave polls one address
// rather than 64, then the missing lanes wait for theirs.  A wave behind the
// frontier pays one memory round trip.  Lanes that want nothing get `empty`.
// `done` is cleared if the wave is to leave its share.
//
// Two forms of the same, since what the compiler makes of a form decides several
// per cent of a sweep's time.  load_or_wait: the required times' (200k cells 97 us,
// 112 by the other); load_or_leave, which returns `done`: the smoothed sums' (1M
// cells 157 + 191 us, 163 + 208 by the other).
template <bool LOW_LAST>
__device__ __forceinline__ int last_missing(int idx, bool miss) {
  return LOW_LAST ? -wave_max_int(miss ? -idx : INT32_MIN + 1) : wave_max_int(miss ? idx : -1);
}
// (each lane in a loop of its own: with Polls::missing 102 us at 200k cells)
template <Sweep S, typename U>
__device__ __forceinline__ U poll_word(const U *p, U empty, int run, const Waits<S> &wt) {
  U u = pub_ld(p);
  int it = 0;
  while (u == empty) {
    if (++it > run) break;
    if ((it & 31) == 0 && pub_ld(&wt.share()->ended) != 0) break;
    __builtin_amdgcn_s_sleep(1);
    u = pub_ld(p);
  }
  return u;
}
// the wait goes on after its first run of polls; returns `done`
template <bool TICKETS, Sweep S, typename U>
__device__ __forceinline__ bool poll_on(const U *p, bool miss, U empty, int run, const Waits<S> &wt, U &v) {
  Polls<TICKETS, S> polls(wt);
  polls.it = run + 1;
  while (polls.resume(miss && v == empty)) {
    do {
      if (miss) v = pub_ld(p);
    } while (polls.missing(miss && v == empty));
  }
  return !polls.leave;
}

template <bool LOW_LAST, bool TICKETS, Sweep S, typename U>
__device__ __forceinline__ U load_or_wait(const U *base, int idx, bool want, U empty, const Waits<S> &wt, bool &done) {
  U v = want ? pub_ld(base + idx) : empty;
  const bool miss = want && v == empty;
  if (__ballot(miss)) {
    const int run = Polls<TICKETS, S>::first_run(wt.limit), rep = last_missing<LOW_LAST>(idx, miss);
    if (wave_lane() == 0) (void)poll_word(base + rep, empty, run, wt);
    if (miss) v = poll_word(base + idx, empty, run, wt);
    if (__ballot(miss && v == empty)) done = poll_on<TICKETS>(base + idx, miss, empty, run, wt, v);
  }
  return v;
}

template <bool LOW_LAST, bool TICKETS, Sweep S, typename U>
__device__ __forceinline__ bool load_or_leave(const U *base, int idx, bool want, U empty, const Waits<S> &wt, U &v) {
  v = want ? pub_ld(base + idx) : empty;
  const bool miss = want && v == empty;
  if (!__ballot(miss)) return true;
  const int rep = last_missing<LOW_LAST>(idx, miss);
  const int run = Polls<TICKETS, S>::first_run(wt.limit);
  auto poll = [&](const U *p) {
    U u = pub_ld(p);
    for (int it = 0; u == empty;) {
      if (++it > run) break;
      if ((it & 31) == 0 && pub_ld(&wt.share()->ended) != 0) break;
      __builtin_amdgcn_s_sleep(1);
      u = pub_ld(p);
    }
    return u;
  };
  if (wave_lane() == 0) (void)poll(base + rep);
  if (miss) v = poll(base + idx);
  if (!__ballot(miss && v == empty)) return true;
  return poll_on<TICKETS>(base + idx, miss, empty, run, wt, v);
}

template <Sweep S>
Waits<S> sweep_waits(tdp_graph g) {
  return Waits<S>{g->sweep_args, g->spin_limit};
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
