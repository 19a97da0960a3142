// One-launch prefix sums and "last workgroup" steps across the workgroups of
// a kernel (decoupled look-back): a workgroup takes the next tile by a ticket,
// publishes its tile's totals, adds up the totals published by the tiles
// before it, and publishes the sum.  Tickets are handed out in order, so the
// lowest tile not yet done is always held by a running workgroup and every
// wait ends; the waits are bounded all the same.  Totals and state share a
// 64-bit word, so no fence is needed, and words carry the launch's number, so
// nothing is cleared between launches.
//
// It replaces a reduce launch and a second pass (and the kernels that made
// and read the flags): a launch behind another costs 2 to 5 us whatever it does.
#pragma once

#include "tdp_wave.h"

namespace tdp {

// st: a state word per tile and value; ctr: {launches so far, ticket, workgroups done}
struct Look {
  uint64_t *st;
  uint32_t *ctr;
  int32_t *err;
};
constexpr int LOOK_MAX = 1 << 22;    // polls per wait

// the workgroup's next tile (>= tiles: none left); every thread gets it
__device__ __forceinline__ int look_tile(const Look &lk) {
  __shared__ int s_tile;
  __syncthreads();
  if (threadIdx.x == 0) s_tile = (int)atomicAdd(lk.ctr + 1, 1u);
  __syncthreads();
  return s_tile;
}

// the tile after `tile`: none when every tile has a workgroup of its own
__device__ __forceinline__ int look_next(const Look &lk, int tiles) {
  return (int)gridDim.x >= tiles ? tiles : look_tile(lk);
}

__device__ __forceinline__ uint64_t look_word(uint32_t launch, uint32_t state, int v) {
  return (uint64_t)(uint32_t)v | (uint64_t)state << 32 | (uint64_t)((launch + 1) & 0x3FFFFFFFu) << 34;
}

// Sum of the totals of the tiles before `tile`; called by one whole wave with
// the tile's totals, `launch` = ctr[0] as read at the kernel's start.
template <int NV>
__device__ __forceinline__ void look_prefix(const Look &lk, int tile, uint32_t launch, const int (&total)[NV],
                                            int (&before)[NV]) {
  const int lane = wave_lane();
  const uint32_t num = (launch + 1) & 0x3FFFFFFFu;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    before[v] = 0;
    if (lane == 0) pub_st(lk.st + (size_t)tile * NV + v, look_word(launch, tile == 0 ? 2 : 1, total[v]));
  }
  if (tile == 0) return;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    int sum = 0;
    for (int end = tile - 1;; end -= 64) {  // 64 tiles at a time, the nearest in lane 0
      const int idx = end - lane;
      uint64_t w = 0;
      bool miss = idx >= 0;
      for (int it = 0; __ballot(miss); ++it) {
        if (miss) {
          w = pub_ld(lk.st + (size_t)idx * NV + v);
          miss = (uint32_t)(w >> 34) != num;
        }
        if (it > LOOK_MAX) {
          if (lane == 0) atomicOr(lk.err, 2);
          break;
        }
      }
      const unsigned long long done = __ballot(idx >= 0 && ((w >> 32) & 3) == 2);
      const int stop = done ? __ffsll((unsigned long long)done) - 1 : 63;  // the nearest tile that knows its prefix
      int x = idx >= 0 && lane <= stop ? (int)(uint32_t)w : 0;
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
      sum += x;
      if (done || end < 64) break;
    }
    before[v] = sum;
    if (lane == 0) pub_st(lk.st + (size_t)tile * NV + v, look_word(launch, 2, sum + total[v]));
  }
}

// every store of this wave has arrived where other workgroups read it (pub_ld)
__device__ __forceinline__ void stores_arrived() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Every workgroup calls it when it is done; true in the last one, which sees
// what the others stored with pub_st, and readies the counters for the next
// launch.
__device__ __forceinline__ bool look_done(const Look &lk, uint32_t launch) {
  __shared__ int s_last;
  stores_arrived();
  __syncthreads();
  if (threadIdx.x == 0) {
    const bool last = atomicAdd(lk.ctr + 2, 1u) == gridDim.x - 1;
    if (last) {
      pub_st(lk.ctr + 1, 0u);
      pub_st(lk.ctr + 2, 0u);
      pub_st(lk.ctr, launch + 1);
    }
    s_last = last;
  }
  __syncthreads();
  return s_last != 0;
}

// doubles that other workgroups of the launch read
__device__ __forceinline__ void pub_st(double *p, double v) {
  pub_st(reinterpret_cast<uint64_t *>(p), (uint64_t)__double_as_longlong(v));
}
__device__ __forceinline__ double pub_ld(const double *p) {
  return __longlong_as_double((long long)pub_ld(reinterpret_cast<const uint64_t *>(p)));
}

// The sum of part[0 .. n) in the last workgroup of a launch to be done, in a
// fixed order, to *out: every workgroup of 256 threads calls it after its
// pub_st of its part.  One launch less per reduction, for launches of some 100
// workgroups: 4,096 that count themselves at one address take 70 us for it.
__device__ __forceinline__ void last_sum(uint32_t *ctr, int n, const double *part, double *out) {
  __shared__ double sh[256];
  if (!look_done(Look{nullptr, ctr, nullptr}, ctr[0])) return;
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) a += pub_ld(part + i);
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

// A barrier among the first `n` workgroups of a launch, all on the GPU at once
// (n is small): every workgroup raises its own flag, and one wave of each
// polls the others' (1 us for up to 32 workgroups; a launch boundary costs 2
// to 5).  Stores made with pub_st before it are seen by pub_ld after it.
// Flags count up over launches and are never cleared: `phase` must be larger at
// every call.  Waits are bounded by `limit` polls: false, with bit 2 of *err set,
// when one ran out; the workgroup then leaves without using what others store.
__device__ __forceinline__ bool group_barrier(uint32_t *flags, int n, uint32_t phase, int32_t *err, int limit) {
  stores_arrived();
  bool out = false;
  __syncthreads();
  if (n > 1 && threadIdx.x < 64) {
    if (threadIdx.x == 0) pub_st(flags + blockIdx.x, phase);
    for (int f = threadIdx.x; f < n; f += 64) {
      int it = 0;
      while ((int)(pub_ld(flags + f) - phase) < 0) {
        if (++it > limit) {
          atomicOr(err, 2);
          out = true;
          break;
        }
      }
    }
  }
  return __syncthreads_or(out) == 0;
}

// exclusive sum of one value per thread over the workgroup (at most 16 waves); total in *total
__device__ __forceinline__ int block_exclusive(int v, int *total) {
  __shared__ int s_wave[17];
  const int lane = wave_lane(), wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  int x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(x, o, 64);
    if (lane >= o) x += u;
  }
  __syncthreads();
  if (lane == 63) s_wave[wid] = x;
  __syncthreads();
  int add = 0, all = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wid) add += s_wave[w];
    all += s_wave[w];
  }
  *total = all;
  return add + x - v;
}

}  // namespace tdp
