// report_timing_endpoint(n, k) on the device (Sec. III-B, Table I).
//
// A path into endpoint e is described by its deviations from the
// arrival-time tree: walking back from e along critical inputs, a deviation
// takes a non-critical input j of a cell instead.  The path's slack is the
// endpoint's slack plus the sum of its deviation costs
//     delta(j) = AT(out) - (AT(in_j) + d_arc(in_j)) >= 0,
// so the k worst paths at e are the k cheapest deviation sets.  Every path has
// a unique parent (itself without its upstream-most deviation) and its children
// add one deviation on the critical chain above that point, so the cheapest
// paths come out of a best-first expansion.  The forward sweep already keeps,
// for every cell, the max_k cheapest deviations along its critical chain, so a
// pop needs one list read, not a chain walk.
//
//   k_sel_*        endpoints of each instance in (slack, pin id) order; the
//                  first n, or the violated ones (n < 0)
//   k_search       KM lanes per selected endpoint: best-first expansion
//                  with the candidate list across the lanes; writes, per path
//                  slot, its slack, its deviation, its parent slot and its pin
//                  count (from the critical-chain depths)
//   ordering       stable radix sort of the slots by (instance, slack); per
//                  instance cut to K; prefix sum of the pin counts
//   k_walk         four lanes per output path: follow critical inputs and
//                  the deviations from the endpoint back to the start point,
//                  writing the pins in place from the end.
#include "tdp_impl.h"
#include "tdp_look.h"
#include "tdp_prims.h"
#include "tdp_walk.h"
#include "tdp_wave.h"

namespace tdp {

// ------------------------------------------------------------- selection
constexpr int SEL_TILE = 4096;  // endpoints per tile: 1024 threads x 4

// The violated endpoints of every instance, in order, in one launch: flags by
// ballot, places by look-back; the place of an instance's first endpoint is
// its inst_selb.  (Five launches, flags through memory, took 21 us at 20,000
// endpoints and 28 at 240,000; this 10 and 12.)
template <typename T>
__global__ void __launch_bounds__(1024) k_sel_violated(Topo tp, Look lk, const int32_t *__restrict__ ep_base,
                                                        const T *__restrict__ ep_slack, int32_t *__restrict__ list,
                                                        int32_t *__restrict__ d_nsel, int32_t *__restrict__ inst_selb) {
  __shared__ unsigned long long s_mask[64];  // rounds x waves
  __shared__ int s_before[64], s_base, s_total;
  const int lane = wave_lane(), wid = threadIdx.x >> 6;
  const uint32_t launch = lk.ctr[0];
  const int tiles = max(1, (tp.E + SEL_TILE - 1) / SEL_TILE);
  for (int tile = look_tile(lk); tile < tiles; tile = look_next(lk, tiles)) {
    const int f0 = tile * SEL_TILE;
    T sl[4];
    unsigned long long m[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int f = f0 + r * 1024 + threadIdx.x;
      sl[r] = f < tp.E ? ep_slack[f] : (T)0;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      m[r] = __ballot(sl[r] < (T)0);
      if (lane == 0) s_mask[r * 16 + wid] = m[r];
    }
    __syncthreads();
    if (wid == 0) {
      const int c = __popcll(s_mask[lane]);
      int x = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(x, o, 64);
        if (lane >= o) x += u;
      }
      s_before[lane] = x - c;
      const int total[1] = {__shfl(x, 63, 64)};
      int before[1];
      look_prefix<1>(lk, tile, launch, total, before);
      if (lane == 0) {
        s_base = before[0];
        s_total = total[0];
      }
    }
    __syncthreads();
    const unsigned long long below = (1ull << lane) - 1;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if ((m[r] >> lane) & 1)
        list[s_base + s_before[r * 16 + wid] + __popcll(m[r] & below)] = f0 + r * 1024 + threadIdx.x;
    const bool last = tile == tiles - 1;
    for (int i = threadIdx.x; i <= tp.num_inst; i += 1024) {
      const int e = ep_base[i] - f0;
      if (e < 0 || (e >= SEL_TILE && !(last && ep_base[i] == tp.E))) continue;
      inst_selb[i] = e >= SEL_TILE ? s_base + s_total
                                   : s_base + s_before[e >> 6] + __popcll(s_mask[e >> 6] & ((1ull << (e & 63)) - 1));
    }
    if (last && threadIdx.x == 0) *d_nsel = s_base + s_total;
  }
  look_done(lk, launch);
}

// The first n endpoints of each instance in (slack, position) order, listed in
// position order: one workgroup per instance holds its keys in registers, R a
// thread, finds the n-th smallest by a radix select (four counts of 8 bits in
// LDS), and lists everything below it and the first of its equals; where its
// part of the list starts comes by look-back.  For instances of up to
// SEL_SELECT endpoints; a sort serves larger ones.  Bound by one workgroup's
// LDS counts and barriers: 15,000 endpoints in 26 us, against 90 by sort,
// flags and scans in some 20 launches (and 60 with the keys read again for
// every count).
constexpr int SEL_SELECT = 1 << 16;
constexpr uint32_t SEL_NEVER = 0xFFFFFFFFu;  // endpoints without a finite slack, never taken

template <typename T>
__device__ __forceinline__ uint32_t sel_key(T slack) {
  return (uint32_t)order_key((float)slack);
}

template <typename T, int R>
__global__ void __launch_bounds__(1024) k_sel_worst(int num_inst, const int32_t *__restrict__ ep_base,
                                                     const T *__restrict__ ep_slack, int n, Look lk,
                                                     int32_t *__restrict__ list, int32_t *__restrict__ d_nsel,
                                                     int32_t *__restrict__ inst_selb) {
  __shared__ int hist[256], s_lt[R * 16], s_eq[R * 16], s_digit, s_below, s_pos;
  const int tid = threadIdx.x, lane = wave_lane(), wid = tid >> 6;
  const unsigned long long below = (1ull << lane) - 1;
  const uint32_t launch = lk.ctr[0];
  for (int inst = look_tile(lk); inst < num_inst; inst = look_next(lk, num_inst)) {
    const int b = ep_base[inst], e = ep_base[inst + 1];
    uint32_t key[R];
    int finite = 0;
#pragma unroll
    for (int r0 = 0; r0 < R; r0 += 16) {
      T sl[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f = b + (r0 + r) * 1024 + tid;
        sl[r] = f < e ? ep_slack[f] : inf_of<T>();
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool in = sl[r] < inf_of<T>();
        key[r0 + r] = in ? sel_key(sl[r]) : SEL_NEVER;
        finite += in;
      }
    }
    int all;
    block_exclusive(finite, &all);
    const int take = min(n, all);
    uint32_t cut = 0;
    int need = take;  // of the endpoints that share the digits settled so far
    if (take > 0) {
      for (int shift = 24; shift >= 0; shift -= 8) {
        if (tid < 256) hist[tid] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < R; ++r)
          if (key[r] != SEL_NEVER && (uint64_t)(key[r] ^ cut) >> (shift + 8) == 0)
            atomicAdd(&hist[(key[r] >> shift) & 255u], 1);
        __syncthreads();
        const int h = tid < 256 ? hist[tid] : 0;
        const int c = block_exclusive(h, &all);
        if (tid < 256 && c < need && c + h >= need) {
          s_digit = tid;
          s_below = c;
        }
        __syncthreads();
        cut |= (uint32_t)s_digit << shift;
        need -= s_below;
      }
    }
    // counts of each 64 endpoints below the cut and at it, to counts before
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int lt = __popcll(__ballot(key[r] < cut)), eq = __popcll(__ballot(key[r] == cut));
      if (lane == 0) {
        s_lt[r * 16 + wid] = lt;
        s_eq[r * 16 + wid] = eq;
      }
    }
    __syncthreads();
    const int lt = block_exclusive(tid < R * 16 ? s_lt[tid] : 0, &all);
    const int eq = block_exclusive(tid < R * 16 ? s_eq[tid] : 0, &all);
    if (tid < R * 16) {
      s_lt[tid] = lt;
      s_eq[tid] = eq;
    }
    if (wid == 0) {
      const int total[1] = {take};
      int before[1];
      look_prefix<1>(lk, inst, launch, total, before);
      if (lane == 0) {
        s_pos = before[0];
        inst_selb[inst] = before[0];
        if (inst == num_inst - 1) *d_nsel = inst_selb[num_inst] = before[0] + take;
      }
    }
    __syncthreads();
    if (take == 0) continue;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool is_lt = key[r] < cut, is_eq = key[r] == cut;
      const unsigned long long ml = __ballot(is_lt), me = __ballot(is_eq);
      const int l = s_lt[r * 16 + wid] + __popcll(ml & below), q = s_eq[r * 16 + wid] + __popcll(me & below);
      if (is_lt || (is_eq && q < need)) list[s_pos + l + min(q, need)] = b + r * 1024 + tid;
    }
  }
  look_done(lk, launch);
}

// larger instances: endpoints taken, the cut's key and its equals among them,
// from the endpoints sorted by (instance, slack, position)
constexpr int SEL_CUT = 4;  // words per instance: the cut's key, endpoints taken, equals taken among them

template <typename T>
__global__ void k_sel_keys(Topo tp, const T *__restrict__ ep_slack, uint64_t *__restrict__ keys,
                           uint32_t *__restrict__ vals) {
  const int f = blockIdx.x * blockDim.x + threadIdx.x;
  if (f >= tp.E) return;
  keys[f] = ((uint64_t)tp.ff_inst[f] << 32) | sel_key(ep_slack[f]);
  vals[f] = f;
}

// first of the ascending keys[0, n) whose low word is >= key, or n: 1,024 places
// looked at per round by the workgroup's 1,024 threads, two or three rounds
__device__ __forceinline__ int block_lower_bound(const uint64_t *__restrict__ keys, int n, uint32_t key) {
  int lo = 0, hi = n;  // the answer lies in [lo, hi]
  while (lo < hi) {
    const int step = (hi - lo + 1023) / 1024, at = lo + (int)threadIdx.x * step;
    const int below = __syncthreads_count(at < hi && (uint32_t)keys[at] < key);  // (the first `below` threads')
    if (below == 0) return lo;
    const int next = lo + (below - 1) * step;
    hi = min(hi, next + step);
    lo = next + 1;
  }
  return lo;
}

// The sorted keys tell where the finite slacks and the cut's equals begin and end
// (a count over the slacks themselves took 143 us of 466 for 140,000 of as many
// endpoints).  A double that rounds to infinity is counted by itself.
template <typename T>
__global__ void __launch_bounds__(1024) k_sel_cut_sorted(const int32_t *__restrict__ ep_base,
                                                          const T *__restrict__ ep_slack,
                                                          const uint64_t *__restrict__ keys,
                                                          const uint32_t *__restrict__ perm, int n,
                                                          int32_t *__restrict__ cut) {
  __shared__ int s_more;
  const int b = ep_base[blockIdx.x], e = ep_base[blockIdx.x + 1];
  if (threadIdx.x == 0) s_more = 0;
  __syncthreads();
  const int m = min(n, e - b);
  const uint32_t inf = (uint32_t)order_key(inf_of<float>());
  // (below minus infinity there are only NaNs)
  const int from = block_lower_bound(keys + b, m, (uint32_t)order_key(-inf_of<float>()));
  const int to = block_lower_bound(keys + b, m, inf);
  if constexpr (sizeof(T) == 8) {
    int c = 0;
    for (int j = to + (int)threadIdx.x; j < m && (uint32_t)keys[b + j] == inf; j += 1024)
      c += ep_slack[perm[b + j]] < inf_of<T>();
    if (c) atomicAdd(&s_more, c);
    __syncthreads();
  }
  const int take = to - from + s_more;
  const uint32_t key = take > 0 ? (uint32_t)keys[b + take - 1] : 0u;
  const int equal = block_lower_bound(keys + b, take, key);
  if (threadIdx.x == 0) {
    cut[SEL_CUT * blockIdx.x] = (int)key;
    cut[SEL_CUT * blockIdx.x + 1] = take;
    cut[SEL_CUT * blockIdx.x + 2] = take - equal;
  }
}

template <typename T>
__global__ void __launch_bounds__(1024) k_sel_take(int num_inst, const int32_t *__restrict__ ep_base,
                                                    const T *__restrict__ ep_slack, const int32_t *__restrict__ cut,
                                                    int32_t *__restrict__ list, int32_t *__restrict__ d_nsel,
                                                    int32_t *__restrict__ inst_selb) {
  __shared__ int s_lt[65], s_eq[65], s_base;
  const int lane = wave_lane(), wid = threadIdx.x >> 6, inst = blockIdx.x;
  if (threadIdx.x == 0) s_base = 0;
  __syncthreads();
  int before = 0;
  for (int i = threadIdx.x; i < inst; i += 1024) before += cut[SEL_CUT * i + 1];
  if (before) atomicAdd(&s_base, before);
  __syncthreads();
  int pos = s_base;
  const uint32_t key = (uint32_t)cut[SEL_CUT * inst];
  const int take = cut[SEL_CUT * inst + 1];
  int equals = cut[SEL_CUT * inst + 2];  // still to take
  if (threadIdx.x == 0) {
    inst_selb[inst] = pos;
    if (inst == num_inst - 1) *d_nsel = inst_selb[num_inst] = pos + take;
  }
  const int b = ep_base[inst], e = ep_base[inst + 1];
  const unsigned long long below = (1ull << lane) - 1;
  if (take == 0) return;
  for (int f0 = b; f0 < e; f0 += 4096) {
    T s[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int f = f0 + r * 1024 + threadIdx.x;
      s[r] = f < e ? ep_slack[f] : inf_of<T>();
    }
    unsigned long long lt[4], eq[4];
    __syncthreads();  // (the masks of the round before are read)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool fin = s[r] < inf_of<T>();
      const uint32_t k = sel_key(s[r]);
      lt[r] = __ballot(fin && k < key);
      eq[r] = __ballot(fin && k == key);
      if (lane == 0) {
        s_lt[r * 16 + wid] = __popcll(lt[r]);
        s_eq[r * 16 + wid] = __popcll(eq[r]);
      }
    }
    __syncthreads();
    if (wid < 2) {  // counts to counts before, over the 64 rounds and waves
      int *c = wid == 0 ? s_lt : s_eq;
      const int v = c[lane];
      int x = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(x, o, 64);
        if (lane >= o) x += u;
      }
      c[lane] = x - v;
      if (lane == 63) c[64] = x;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int l = s_lt[r * 16 + wid] + __popcll(lt[r] & below), q = s_eq[r * 16 + wid] + __popcll(eq[r] & below);
      const bool in = ((lt[r] >> lane) & 1) || (((eq[r] >> lane) & 1) && q < equals);
      if (in) list[pos + l + min(q, equals)] = f0 + r * 1024 + threadIdx.x;
    }
    const int qall = min(s_eq[64], equals);
    pos += s_lt[64] + qall;
    equals -= qall;
  }
}

// --------------------------------------------------------------- search
// KM lanes per selected endpoint.  Lane j holds candidate j of the list of
// unpopped paths (ascending by cost, then creation order) and, once found,
// path j.  A pop reads the deviation list of the popped path's chain start,
// lane j its entry j, and merges the two sorted lists by rank through LDS, so a
// pop costs its two dependent loads (the deviation's driver, then the list)
// and some 4 KM instructions.  One thread per endpoint with the lists in
// registers took KM^2 dependent steps per pop and left most of the chip
// idle: 78 us against 18 for 1,000 endpoints at k = 10, KM = 16; 28 against 18
// for 12,000 at k = KM = 8.
template <typename T, int KM>
__global__ void __launch_bounds__(64) k_search(Topo tp, int k, T slack_limit, const int32_t *__restrict__ d_nsel,
                                                const int32_t *__restrict__ sel, const T *__restrict__ ep_slack,
                                                const uint32_t *__restrict__ cdep, const uint64_t *__restrict__ node,
                                                T *__restrict__ slot_key,
                                                int32_t *__restrict__ slot_dev, int32_t *__restrict__ slot_par,
                                                int32_t *__restrict__ slot_len) {
  static_assert(KM >= 1 && KM <= 32 && (KM & (KM - 1)) == 0, "a power of two of at most half a wave");
  __shared__ T s_cost[64];
  __shared__ int32_t s_dev[64], s_par[64];
  const int lane = threadIdx.x, j = lane & (KM - 1), base = lane & ~(KM - 1);
  const int nsel = *d_nsel;
  if (blockIdx.x * (64 / KM) >= nsel) return;  // whole wave: the grid is sized for every endpoint
  const int q = blockIdx.x * (64 / KM) + lane / KM;
  bool live = q < nsel;
  const int f = sel[live ? q : nsel - 1];
  const T se = ep_slack[f];
  const int eroot = tp.snk_drv[tp.A + f];
  // candidates: the endpoint's critical path alone
  T cc = j == 0 ? (T)0 : inf_of<T>();
  int cdv = -1, cpr = -1;
  T okey = inf_of<T>();
  int odev = -1, opar = -1, ocells = 0;
  int npop = 0;
  s_cost[lane] = inf_of<T>();
  s_dev[lane] = -1;
  s_par[lane] = -1;
  for (int r = 0; r < k && r < KM; ++r) {
    // pop
    const T cost = __shfl(cc, base, 64);
    const int dev = __shfl(cdv, base, 64), par = __shfl(cpr, base, 64);
    const T sk = se + cost;
    live = live && cost < inf_of<T>() && sk < slack_limit;
    if (!__ballot(live)) break;
    {
      const T nc = __shfl_down(cc, 1, KM);
      const int nd = __shfl_down(cdv, 1, KM), np = __shfl_down(cpr, 1, KM);
      cc = j + 1 < KM ? nc : inf_of<T>();
      cdv = j + 1 < KM ? nd : -1;
      cpr = j + 1 < KM ? np : -1;
    }
    // its chain start and number of cells
    int u = eroot, dc = 0;
    if (live && dev >= 0) {
      u = tp.snk_drv[dev];
      dc = tp.snk_comb[dev];
    }
    const int pc = __shfl(ocells, base + (par >= 0 ? par : 0), 64);
    // children: one more deviation on the critical chain above u
    T d = inf_of<T>();
    int32_t p = -1;
    int cells = 0;
    if (live) {
      const bool more = r + 1 < k && u >= tp.n_start;
      if constexpr (KM > 1) {
        if (more) {
          const Dev<T> e = list_entry<T, KM>(node, u - tp.n_start, j);
          d = e.cost;
          p = e.sink;
        }
      }
      cells = (int)(cdep[u] & ID_MASK);
      if (dev >= 0) cells += pc + 1 - (int)(cdep[tp.n_start + dc] & ID_MASK);
      cells = min(max(cells, 0), tp.D);  // (out of range only after a failed update)
    }
    if (live && j == r) {
      okey = sk;
      odev = dev;
      opar = par;
      ocells = cells;
    }
    npop += live;
    if constexpr (KM > 1) {
      const T ch = d < inf_of<T>() ? cost + d : inf_of<T>();
      // ranks in the merged list: a child goes behind every candidate of
      // equal cost (they were created earlier)
      int rc = j, rd = j;
#pragma unroll
      for (int i = 0; i < KM; ++i) {
        rc += __shfl(ch, base + i, 64) < cc;
        rd += !(ch < __shfl(cc, base + i, 64));
      }
      if (rc < KM) {
        s_cost[base + rc] = cc;
        s_dev[base + rc] = cdv;
        s_par[base + rc] = cpr;
      }
      if (rd < KM) {
        s_cost[base + rd] = ch;
        s_dev[base + rd] = p;
        s_par[base + rd] = r;
      }
      __syncthreads();
      cc = s_cost[lane];
      cdv = s_dev[lane];
      cpr = s_par[lane];
      __syncthreads();
    }
  }
  if (q >= nsel || j >= k) return;
  const size_t o = (size_t)q * k + j;
  slot_key[o] = okey;
  slot_dev[o] = odev;
  slot_par[o] = opar;
  slot_len[o] = j < npop ? 2 * ocells + 2 : 0;
}

// ------------------------------------------------------------- ordering
// Slots are ordered by (instance, slack, slot); the first K found ones of an
// instance are its paths.  inst_selb gives each instance's first slot.
template <typename T>
__device__ __forceinline__ uint64_t slot_order(const Topo &tp, int f, T key) {
  if constexpr (sizeof(T) == 4) return ((uint64_t)tp.ff_inst[f] << 32) | (order_key((float)key) & 0xFFFFFFFFull);
  else return order_key((double)key);
}

template <typename T>
__global__ void k_slot_keys(Topo tp, int k, const int32_t *__restrict__ d_nsel, const int32_t *__restrict__ sel,
                            const T *__restrict__ slot_key, int32_t *__restrict__ d_nslots,
                            uint64_t *__restrict__ keys, uint32_t *__restrict__ vals) {
  const int n = *d_nsel * k, nth = gridDim.x * blockDim.x;
  const int i0 = blockIdx.x * blockDim.x + threadIdx.x;
  if (i0 == 0) *d_nslots = n;
  for (int i = i0; i < n; i += nth) {
    keys[i] = slot_order<T>(tp, sel[i / k], slot_key[i]);
    vals[i] = (uint32_t)i;
  }
}

// The whole ordering in one launch, single precision: a stable radix sort of
// {instance, slack, slot} words by instance and slack, then the output index
// and first pin of every path.  One workgroup per 2,048 live slots (known on
// the device only), at most ORDER_GROUPS; the others of the grid leave at
// once.  A workgroup owns a run of slots, a wave a run of those: pass by pass
// (8 bits) every wave ranks its words against its own counters in LDS, the
// workgroup publishes its digits' counts, and after a barrier finds their
// places from everyone's counts and moves its words.  What workgroups exchange
// goes through device-scope stores and loads.  Bound by the barriers (two a
// pass) and the round trips around them.  10,000 slots (200k cells): 50 us,
// against 65 in nine launches and 103 in 22 (and 85 with 11-bit digits: more to
// clear, add up and read per pass than a pass saves); 96,000 (2M cells): 86
// against 115 in eleven launches.  Without passes, behind k_rank: 12 us for 10,000.
constexpr int ORDER_GROUPS = 64;
constexpr int ORDER_ITEMS = 2;  // words per thread and round
constexpr int ORDER_RUN = 1024 * ORDER_ITEMS;

struct OrderBuf {
  uint64_t *w0, *w1;
  uint32_t *hist;   // [ORDER_GROUPS][256]
  uint64_t *total;  // [ORDER_GROUPS] kept slots and their pins
  uint32_t *flags;  // [ORDER_GROUPS] barrier flags, then the phase that the launch's barriers count up from
  int limit;        // polls per wait
};
// phases per launch at most: a barrier more than two a pass of 8 bits
constexpr uint32_t ORDER_PHASES = 32;

// Slots of instances that have at most RANK_MOST each are put in order by
// counting, for every slot, the slots of its instance that come before it: no
// pass waits for another, and the compute units share the comparisons (10,000
// slots: 10^8 in 21 us, where k_order's passes take 38).  One workgroup per
// 64 slots, a lane each; its 16 waves count a part of every tile of keys in LDS.
constexpr int RANK_MOST = 1 << 14;
constexpr int RANK_TILE = 4096;

// whether counting orders this call's slots (the same answer in every thread
// of every workgroup)
__device__ __forceinline__ bool rank_orders(int num_inst, int k, const int32_t *__restrict__ inst_selb) {
  bool big = false;
  for (int i = threadIdx.x; i < num_inst; i += blockDim.x)
    big = big || (long long)(inst_selb[i + 1] - inst_selb[i]) * k > RANK_MOST;
  return __syncthreads_or(big) == 0;
}

__global__ void __launch_bounds__(1024) k_rank(Topo tp, int k, int slot_bits, const int32_t *__restrict__ d_nsel,
                                                const int32_t *__restrict__ sel, const int32_t *__restrict__ inst_selb,
                                                const float *__restrict__ slot_key, uint64_t *__restrict__ words,
                                                uint32_t *__restrict__ order_phase) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *order_phase += ORDER_PHASES;  // (k_order's, which is next)
  __shared__ uint4 s_key[RANK_TILE / 4];
  __shared__ int s_cnt[16][64];
  const int n = *d_nsel * k;
  if ((int)blockIdx.x * 64 >= n || !rank_orders(tp.num_inst, k, inst_selb)) return;
  const int lane = wave_lane(), wid = threadIdx.x >> 6;
  for (int e0 = blockIdx.x * 64; e0 < n; e0 += gridDim.x * 64) {
    const int i = min(e0 + lane, n - 1);
    const int inst = tp.ff_inst[sel[i / k]];
    const int s0 = inst_selb[inst] * k, s1 = inst_selb[inst + 1] * k;  // the lane's instance's slots
    const uint64_t word = slot_order<float>(tp, sel[i / k], slot_key[i]);
    const uint32_t key = (uint32_t)word;
    const int a = __shfl(s0, 0, 64), z = __shfl(s1, 63, 64);  // of all the lanes' instances
    const bool one = __shfl(s1, 0, 64) == z;
    int count = 0;
    for (int t0 = a; t0 < z; t0 += RANK_TILE) {
      float raw[RANK_TILE / 1024];
#pragma unroll
      for (int r = 0; r < RANK_TILE / 1024; ++r) raw[r] = slot_key[min(t0 + r * 1024 + (int)threadIdx.x, z - 1)];
      __syncthreads();
#pragma unroll
      for (int r = 0; r < RANK_TILE / 1024; ++r) {
        const int j = r * 1024 + (int)threadIdx.x;  // (past the end: before nothing)
        reinterpret_cast<uint32_t *>(s_key)[j] = t0 + j < z ? (uint32_t)order_key(raw[r]) : 0xFFFFFFFFu;
      }
      __syncthreads();
      // this wave's part of the tile: before the workgroup's own slots, after them, or neither
      const int j0 = wid * (RANK_TILE / 16), j1 = min(j0 + RANK_TILE / 16, z - t0);
      if (one && t0 + j1 <= e0) {
#pragma unroll 4
        for (int j = j0; j < j1; j += 4) {
          const uint4 v = s_key[j / 4];
          count += (v.x <= key) + (v.y <= key) + (v.z <= key) + (v.w <= key);
        }
      } else if (one && t0 + j0 >= e0 + 64) {
#pragma unroll 4
        for (int j = j0; j < j1; j += 4) {
          const uint4 v = s_key[j / 4];
          count += (v.x < key) + (v.y < key) + (v.z < key) + (v.w < key);
        }
      } else {
        const uint32_t *ks = reinterpret_cast<const uint32_t *>(s_key);
        const int m0 = one ? max(j0, min(e0 - t0, j1)) : j0, m1 = one ? max(j0, min(e0 + 64 - t0, j1)) : j1;
#pragma unroll 8
        for (int j = j0; j < m0; ++j) count += ks[j] <= key;
#pragma unroll 8
        for (int j = m0; j < m1; ++j) {
          const uint32_t kj = ks[j];
          const int at = t0 + j;
          count += (at >= s0) & (at < s1) & ((kj < key) | ((kj == key) & (at < i)));
        }
#pragma unroll 8
        for (int j = max(m1, j0); j < j1; ++j) count += ks[j] < key;
      }
    }
    __syncthreads();
    s_cnt[wid][lane] = count;
    __syncthreads();
    if (wid == 0 && e0 + lane < n) {
      int rank = 0;
#pragma unroll
      for (int w = 0; w < 16; ++w) rank += s_cnt[w][lane];
      words[s0 + rank] = word << slot_bits | (uint64_t)i;
    }
  }
}

__global__ void __launch_bounds__(1024) k_order(Topo tp, int k, int K, int key_bits, int slot_bits,
                                                 const int32_t *__restrict__ d_nsel, const int32_t *__restrict__ sel,
                                                 const int32_t *__restrict__ inst_selb,
                                                 const float *__restrict__ slot_key,
                                                 const int32_t *__restrict__ slot_len, OrderBuf ob,
                                                 int32_t *__restrict__ d_nslots, int32_t *__restrict__ out_slot,
                                                 int32_t *__restrict__ slot_out, int32_t *__restrict__ path_ptr,
                                                 int32_t *__restrict__ d_num_paths, int32_t *__restrict__ err) {
  constexpr int WAVES = 16;
  __shared__ uint32_t cnt[WAVES][256], s_base[256];
  const int tid = threadIdx.x, lane = wave_lane(), wid = tid >> 6, me = blockIdx.x;
  const int n = *d_nsel * k;
  const int groups = min((int)gridDim.x, max(1, (n + ORDER_RUN - 1) / ORDER_RUN));
  if (me >= groups) return;
  uint32_t phase = ob.flags[ORDER_GROUPS];
  // this workgroup's slots, and this wave's, in rounds of ORDER_ITEMS words a lane
  const int run = ((n + groups - 1) / groups + ORDER_RUN - 1) / ORDER_RUN * ORDER_RUN;
  const int b = min(n, me * run), e = min(n, b + run);
  const int wrun = run / WAVES;
  const int wb = min(e, b + wid * wrun), we = min(e, wb + wrun);
  const bool single = run == ORDER_RUN;  // the words of a round stay in registers
  const uint64_t slot_mask = (1ull << slot_bits) - 1;
  const unsigned long long below = (1ull << lane) - 1;
  uint64_t *wa = ob.w0, *wz = ob.w1;
  const int passes = rank_orders(tp.num_inst, k, inst_selb) ? 0 : (key_bits + 7) / 8;  // 0: k_rank put them in order
  for (int pass = 0; pass < passes; ++pass) {
    const int shift = slot_bits + 8 * pass;
    uint64_t ww[ORDER_ITEMS];
    auto load = [&](int i0) {
#pragma unroll
      for (int j = 0; j < ORDER_ITEMS; ++j) {
        const int i = i0 + j * 64 + lane;
        ww[j] = 0;
        if (i < we)
          ww[j] = pass == 0 ? slot_order<float>(tp, sel[i / k], slot_key[i]) << slot_bits | (uint64_t)i : pub_ld(wa + i);
      }
    };
    // the lanes of the round's j-th word that share this lane's digit
    auto peers = [&](int i0, int j, uint32_t &d) {
      d = (uint32_t)(ww[j] >> shift) & 255u;
      uint64_t m = __ballot(i0 + j * 64 + lane < we);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const uint64_t bal = __ballot((d >> q) & 1u);
        m &= ((d >> q) & 1u) ? bal : ~bal;
      }
      return m;
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) cnt[wid][q * 64 + lane] = 0;
    for (int i0 = wb; i0 < we; i0 += 64 * ORDER_ITEMS) {
      load(i0);
#pragma unroll
      for (int j = 0; j < ORDER_ITEMS; ++j) {
        uint32_t d;
        const uint64_t m = peers(i0, j, d);
        if (((m >> lane) & 1) && (m & below) == 0) cnt[wid][d] += (uint32_t)__popcll(m);
      }
    }
    __syncthreads();
    // counts to places among the waves; the sums to everyone
    uint32_t mine = 0;
    if (tid < 256) {
      uint32_t c[WAVES];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) c[w] = cnt[w][tid];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        cnt[w][tid] = mine;
        mine += c[w];
      }
      if (groups > 1) pub_st(ob.hist + me * 256 + tid, mine);
    }
    if (!group_barrier(ob.flags, groups, ++phase, err, ob.limit)) return;
    uint32_t before = 0, total = mine;
    if (tid < 256 && groups > 1) {
      total = 0;
#pragma unroll 16
      for (int g = 0; g < groups; ++g) {
        const uint32_t h = pub_ld(ob.hist + g * 256 + tid);
        total += h;
        before += g < me ? h : 0u;
      }
    }
    int all;
    const uint32_t base = (uint32_t)block_exclusive((int)total, &all);
    if (tid < 256) s_base[tid] = base + before;
    __syncthreads();
    for (int i0 = wb; i0 < we; i0 += 64 * ORDER_ITEMS) {
      if (!single) load(i0);
#pragma unroll
      for (int j = 0; j < ORDER_ITEMS; ++j) {
        uint32_t d;
        const uint64_t m = peers(i0, j, d);
        const uint32_t place = cnt[wid][d];
        if ((m >> lane) & 1) {
          pub_st(wz + s_base[d] + place + __popcll(m & below), ww[j]);
          if ((m & below) == 0) cnt[wid][d] = place + (uint32_t)__popcll(m);
        }
      }
    }
    if (!group_barrier(ob.flags, groups, ++phase, err, ob.limit)) return;
    uint64_t *t = wa;
    wa = wz;
    wz = t;
  }
  // kept slots, in order: the first K found ones of their instance
  const uint64_t inf_key = order_key(inf_of<float>());
  auto kept = [&](int j, int &slot, int &len) {
    const uint64_t w = pub_ld(wa + j), key = w >> slot_bits;
    slot = (int)(w & slot_mask);
    const bool in = (key & 0xFFFFFFFFull) < inf_key && j - inst_selb[(int)(key >> 32)] * k < K;
    len = in ? slot_len[slot] : 0;
    return in;
  };
  int paths = 0, pins = 0;  // of the workgroup's run, this thread's share
  for (int j0 = b; j0 < e; j0 += 1024) {
    int slot, len = 0;
    if (j0 + tid < e) paths += kept(j0 + tid, slot, len);
    pins += len;
  }
  int q0 = 0, p0 = 0;
  if (groups > 1) {
    int c, p;
    block_exclusive(paths, &c);
    block_exclusive(pins, &p);
    if (tid == 0) pub_st(ob.total + me, (uint64_t)(uint32_t)c | (uint64_t)(uint32_t)p << 32);
    if (!group_barrier(ob.flags, groups, ++phase, err, ob.limit)) return;
    for (int g = 0; g < me; ++g) {
      const uint64_t w = pub_ld(ob.total + g);
      q0 += (int)(uint32_t)w;
      p0 += (int)(uint32_t)(w >> 32);
    }
  }
  for (int j0 = b; j0 < e; j0 += 1024) {
    int slot = 0, len = 0, c, p;
    const bool on = j0 + tid < e && kept(j0 + tid, slot, len);
    const int q = q0 + block_exclusive(on, &c), at = p0 + block_exclusive(len, &p);
    if (j0 + tid < e) slot_out[slot] = on ? q : -1;
    if (on) {
      out_slot[q] = slot;
      path_ptr[q] = at;
    }
    q0 += c;
    p0 += p;
  }
  if (me == groups - 1 && tid == 0) {
    *d_nslots = n;
    *d_num_paths = q0;
    path_ptr[q0] = p0;
  }
}

// the same steps as launches of their own, where a slot's word does not fit
// 64 bits (double precision; hundreds of instances with many slots): output
// index and first pin of every path from the sorted slots, summed together by
// look-back
constexpr int OUT_TILE = 2048;  // 256 threads x 8

template <typename T>
__global__ void __launch_bounds__(256) k_path_out(int k, int K, Look lk, const int32_t *__restrict__ d_nslots,
                                                   const int32_t *__restrict__ inst_selb,
                                                   const uint64_t *__restrict__ keys, const uint32_t *__restrict__ perm,
                                                   const int32_t *__restrict__ slot_len, int32_t *__restrict__ out_slot,
                                                   int32_t *__restrict__ slot_out, int32_t *__restrict__ path_ptr,
                                                   int32_t *__restrict__ d_num_paths) {
  __shared__ int s_base[2];
  const uint32_t launch = lk.ctr[0];
  const int n = *d_nslots;
  const int tiles = max(1, (n + OUT_TILE - 1) / OUT_TILE);
  const uint64_t inf_key = sizeof(T) == 4 ? order_key(inf_of<float>()) : order_key(inf_of<double>());
  for (int tile = look_tile(lk); tile < tiles; tile = look_next(lk, tiles)) {
    const int j0 = tile * OUT_TILE + threadIdx.x * 8;
    int slot[8], len[8];
    bool kept[8];
    int cnt = 0, pins = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int j = j0 + q;
      const uint64_t key = j < n ? keys[j] : inf_key;
      slot[q] = j < n ? (int)perm[j] : 0;
      const int inst = sizeof(T) == 4 && j < n ? (int)(key >> 32) : 0;
      kept[q] = j < n && (sizeof(T) == 4 ? (key & 0xFFFFFFFFull) : key) < inf_key && j - inst_selb[inst] * k < K;
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      len[q] = kept[q] ? slot_len[slot[q]] : 0;
      cnt += kept[q];
      pins += len[q];
    }
    int total[2], before[2];
    int c = block_exclusive(cnt, &total[0]), p = block_exclusive(pins, &total[1]);
    if (threadIdx.x < 64) {
      look_prefix<2>(lk, tile, launch, total, before);
      if (threadIdx.x == 0) {
        s_base[0] = before[0];
        s_base[1] = before[1];
      }
    }
    __syncthreads();
    c += s_base[0];
    p += s_base[1];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (j0 + q >= n) break;
      slot_out[slot[q]] = kept[q] ? c : -1;
      if (kept[q]) {
        out_slot[c] = slot[q];
        path_ptr[c] = p;
        ++c;
        p += len[q];
      }
    }
    if (tile == tiles - 1 && threadIdx.x == 0) {
      *d_num_paths = s_base[0] + total[0];
      path_ptr[s_base[0] + total[0]] = s_base[1] + total[1];
    }
  }
  look_done(lk, launch);
}

// The whole ordering in one workgroup, for at most ORDER_ONE slots: a bitonic
// sort of {instance, slack, slot} words in LDS, then the output indices.  9 us
// for 100 slots (22 launches of 2 us before); with 7,000 it took 82.
constexpr int ORDER_ONE = 2048;
constexpr int ORDER_SLOT_BITS = 11;

__global__ void __launch_bounds__(1024) k_order_one(Topo tp, int k, int K, const int32_t *__restrict__ d_nsel,
                                                     const int32_t *__restrict__ sel,
                                                     const int32_t *__restrict__ inst_selb,
                                                     const float *__restrict__ slot_key,
                                                     const int32_t *__restrict__ slot_len,
                                                     int32_t *__restrict__ d_nslots, int32_t *__restrict__ out_slot,
                                                     int32_t *__restrict__ slot_out, int32_t *__restrict__ path_ptr,
                                                     int32_t *__restrict__ d_num_paths) {
  __shared__ uint64_t s_key[ORDER_ONE];
  const int n = min(*d_nsel * k, ORDER_ONE);
  int m = 64;
  while (m < n) m <<= 1;
  for (int i = threadIdx.x; i < m; i += 1024)
    s_key[i] = i < n ? slot_order<float>(tp, sel[i / k], slot_key[i]) << ORDER_SLOT_BITS | (uint64_t)i : ~0ull;
  __syncthreads();
  for (int size = 2; size <= m; size <<= 1) {
    for (int d = size >> 1; d > 0; d >>= 1) {
      for (int q = threadIdx.x; q < m / 2; q += 1024) {
        const int i = 2 * q - (q & (d - 1));  // the pair (i, i + d)
        const uint64_t a = s_key[i], b = s_key[i + d];
        if ((a > b) == ((i & size) == 0)) {
          s_key[i] = b;
          s_key[i + d] = a;
        }
      }
      __syncthreads();
    }
  }
  // consecutive slots per thread
  const uint64_t inf_key = order_key(inf_of<float>());
  int len[ORDER_ONE / 1024];
  int cnt = 0, pins = 0;
  const int per = (m + 1023) / 1024, j0 = threadIdx.x * per;
#pragma unroll
  for (int q = 0; q < ORDER_ONE / 1024; ++q) {
    const int j = j0 + q;
    len[q] = -1;
    if (q >= per || j >= n) continue;
    const uint64_t key = s_key[j] >> ORDER_SLOT_BITS;
    if ((key & 0xFFFFFFFFull) < inf_key && j - inst_selb[(int)(key >> 32)] * k < K) {
      len[q] = slot_len[s_key[j] & (ORDER_ONE - 1)];
      ++cnt;
      pins += len[q];
    }
  }
  int all, all_pins;
  int c = block_exclusive(cnt, &all), p = block_exclusive(pins, &all_pins);
#pragma unroll
  for (int q = 0; q < ORDER_ONE / 1024; ++q) {
    const int j = j0 + q;
    if (q >= per || j >= n) continue;
    const int slot = (int)(s_key[j] & (ORDER_ONE - 1));
    slot_out[slot] = len[q] >= 0 ? c : -1;
    if (len[q] >= 0) {
      out_slot[c] = slot;
      path_ptr[c] = p;
      ++c;
      p += len[q];
    }
  }
  if (threadIdx.x == 0) {
    *d_nslots = n;
    *d_num_paths = all;
    path_ptr[all] = all_pins;
  }
}

// ----------------------------------------------------------------- walk
// Four lanes per path, one per hop of a node record: a step loads the record
// of the path's current cell, 16 bytes a lane, and moves the path four cells
// on (fewer at a deviation or at the start point); each lane writes its hop's
// two pins in place, 32 bytes of each output array per path and step.  The
// path's deviations are gathered first, with all that a step needs of them, so
// the record is the step's only load.  Bound by the chain of records (a quarter
// of the path's cells) and, with many paths, by the writes.  A lane per path
// that staged its pins in LDS spent most of a step on its eight pins one
// after another: 53 us against 18 for 10,000 paths at 200k cells, 105 against
// 95 for 96,000 at 2M.
constexpr int WALK_PATHS = 32;  // per workgroup of 128

template <typename T>
__global__ void __launch_bounds__(128) k_walk(Topo tp, int k, int32_t *__restrict__ d_num_paths,
                                               const int32_t *__restrict__ out_slot, const int32_t *__restrict__ sel,
                                               const int32_t *__restrict__ slot_dev, const int32_t *__restrict__ slot_par,
                                               const T *__restrict__ slot_key, const uint64_t *__restrict__ node,
                                               int words, int32_t *__restrict__ path_ptr,
                                               int32_t *__restrict__ path_pins, int32_t *__restrict__ path_int,
                                               int32_t *__restrict__ path_ep, int32_t *__restrict__ path_epi,
                                               int32_t *__restrict__ path_rank, T *__restrict__ path_slack,
                                               int32_t *__restrict__ err, int pin_cap, int32_t *__restrict__ d_nslots) {
  // after a wait that ran out the order may be of several calls: no paths, and
  // reading them reports it
  if (*err & 2) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *d_num_paths = *d_nslots = path_ptr[0] = 0;
    return;
  }
  // a deviation: its sink, cell, driver and both external ids
  __shared__ int32_t s_dev[WALK_PATHS][TDP_MAX_K][5];
  const int lane = wave_lane(), h = lane & 3, first = lane & ~3, mine = threadIdx.x >> 2;
  const int q = blockIdx.x * WALK_PATHS + mine;
  const int n = *d_num_paths;
  if ((int)blockIdx.x * WALK_PATHS >= n) return;
  bool live = q < n;
  int slot = 0, r = 0, f = 0, lo = 0, hi = 0, nd = 0;
  if (live) {
    slot = out_slot[q];
    const int qs = slot / k;
    r = slot - qs * k;
    f = sel[qs];
    lo = path_ptr[q];
    hi = path_ptr[q + 1];
    // deviations, upstream-most first (the walk meets them last to first)
    for (int a = r; a >= 0 && nd < TDP_MAX_K;) {
      const int d = slot_dev[qs * k + a];
      if (d < 0) break;
      if (h == 0) s_dev[mine][nd][0] = d;
      ++nd;
      a = slot_par[qs * k + a];
    }
    if (lo < 0 || hi > pin_cap || hi - lo < 2) {  // only after a failed update
      if (h == 0) atomicOr(err, 1);
      live = false;
    }
  }
  __syncthreads();
  if (live) {
    for (int i = h; i < nd; i += 4) {
      const int d = s_dev[mine][i][0], drv = tp.snk_drv[d];
      s_dev[mine][i][1] = tp.snk_comb[d];
      s_dev[mine][i][2] = drv;
      s_dev[mine][i][3] = tp.snk_ext[d];
      s_dev[mine][i][4] = tp.drv_ext[drv];
    }
  }
  __syncthreads();
  const int et = tp.A + f;
  int v = 0, pos = 0, di = nd - 1;
  // two pins at pos - 1 (driver) and pos (sink); path ranges start at even positions
  auto put = [&](int at, int drv, int drv_ext, int snk, int snk_ext) {
    *(int2 *)(path_pins + at - 1) = make_int2(drv_ext, snk_ext);
    *(int2 *)(path_int + at - 1) = make_int2(drv, tp.M + snk);
  };
  if (live) {
    v = tp.snk_drv[et];
    pos = hi - 1;
    if (h == 0) put(pos, v, tp.drv_ext[v], et, tp.snk_ext[et]);
    pos -= 2;
  }
  for (;;) {
    const bool go = live && v >= tp.n_start && pos > lo;
    if (!__ballot(go)) break;
    int4 rec = make_int4(0, -1, 0, 0);
    if (go) rec = reinterpret_cast<const int4 *>(node + (size_t)(v - tp.n_start) * words)[h];
    // the driver this lane's hop starts at, and whether the chain gets there
    const int up = __shfl_up(rec.y, 1, 4);
    const int at = h == 0 ? v : up;
    const bool there = go && at >= tp.n_start;
    const unsigned on = (unsigned)(__ballot(there) >> first) & 15u;
    const int dc = di >= 0 ? s_dev[mine][di][1] : -1;
    const unsigned hit = (unsigned)(__ballot(there && at - tp.n_start == dc) >> first) & 15u;
    // hops before the first one the chain does not reach, up to and with a deviation
    int hops = __ffs(~on & 31u) - 1;
    const int dev = hit ? __ffs(hit) - 1 : 4;
    const bool turn = dev < hops;
    if (turn) hops = dev + 1;
    int snk = id30((uint32_t)rec.x), drv = rec.y, snk_ext = (int)((uint32_t)rec.z & ID_MASK), drv_ext = rec.w;
    if (turn && h == dev) {
      const int32_t *s = s_dev[mine][di];
      snk = s[0];
      drv = s[2];
      snk_ext = s[3];
      drv_ext = s[4];
    }
    const int p = pos - 2 * h;
    if (go && h < hops && p > lo) put(p, drv, drv_ext, snk, snk_ext);
    const int nv = __shfl(drv, first + (hops > 0 ? hops - 1 : 0), 64);
    if (go) {
      v = nv;
      pos -= 2 * hops;
      if (turn) --di;
    }
  }
  if (!live || h != 0) return;
  if (pos != lo - 1 || v >= tp.n_start || di >= 0) atomicOr(err, 1);
  path_ep[q] = tp.snk_ext[et];
  path_epi[q] = f;
  path_rank[q] = r;
  path_slack[q] = slot_key[slot];
}

// path_ptr[num_paths] = path_ptr[num_paths-1] + len (the scan is exclusive)
__global__ void k_ptr_tail(const int32_t *__restrict__ d_num_paths, const int32_t *__restrict__ len,
                           int32_t *__restrict__ ptr) {
  const int n = *d_num_paths;
  ptr[n] = n > 0 ? ptr[n - 1] + len[n - 1] : 0;
}

// ------------------------------------------------------------- launcher
static inline int nb(long long n, int b) { return n > 0 ? (int)((n + b - 1) / b) : 1; }

template <typename T, int KM>
static void launch_search(tdp_graph g, int k, T limit, hipStream_t s) {
  const Topo &tp = g->topo;
  hipLaunchKernelGGL((k_search<T, KM>), dim3(nb(tp.E, 64 / KM)), dim3(64), 0, s, tp, k, limit, g->d_nsel, g->sel_list,
                     (const T *)g->ep_slack, g->cdep, g->node, (T *)g->slot_key,
                     g->slot_dev, g->slot_par, g->slot_len);
}

// endpoints of each instance: the first n in (slack, pin) order, or the
// violated ones (n < 0); fills sel_list, d_nsel and inst_selb
template <typename T>
void select_stage(tdp_graph g, int n, hipStream_t s) {
  const Topo &tp = g->topo;
  const int E = tp.E;
  const Look lk{g->look_st, g->look_ctr, g->d_err};
  if (n < 0) {
    hipLaunchKernelGGL(k_sel_violated<T>, dim3(std::min(512, nb(E, SEL_TILE))), dim3(1024), 0, s, tp, lk, g->d_ep_base,
                       (const T *)g->ep_slack, g->sel_list, g->d_nsel, g->inst_selb);
    return;
  }
  int most = 0;
  for (int i = 0; i < tp.num_inst; ++i) most = std::max(most, g->lv.ep_base[i + 1] - g->lv.ep_base[i]);
  if (most <= SEL_SELECT) {
    const dim3 grid(std::min(256, tp.num_inst));
    if (most <= 16 * 1024)
      hipLaunchKernelGGL((k_sel_worst<T, 16>), grid, dim3(1024), 0, s, tp.num_inst, g->d_ep_base,
                         (const T *)g->ep_slack, n, lk, g->sel_list, g->d_nsel, g->inst_selb);
    else
      hipLaunchKernelGGL((k_sel_worst<T, 64>), grid, dim3(1024), 0, s, tp.num_inst, g->d_ep_base,
                         (const T *)g->ep_slack, n, lk, g->sel_list, g->d_nsel, g->inst_selb);
    return;
  }
  hipLaunchKernelGGL(k_sel_keys<T>, dim3(nb(E, 256)), dim3(256), 0, s, tp, (const T *)g->ep_slack, g->sort_k0,
                     g->sort_v0);
  const Sorted<uint64_t> so = radix_sort(g->sort_k0, g->sort_v0, g->sort_k1, g->sort_v1, E, nullptr, g->key_bits32, 11,
                                         g->sort_hist, s);
  hipLaunchKernelGGL(k_sel_cut_sorted<T>, dim3(tp.num_inst), dim3(1024), 0, s, g->d_ep_base, (const T *)g->ep_slack,
                     so.keys, so.vals, n, g->sel_cut);
  hipLaunchKernelGGL(k_sel_take<T>, dim3(tp.num_inst), dim3(1024), 0, s, tp.num_inst, g->d_ep_base,
                     (const T *)g->ep_slack, g->sel_cut, g->sel_list, g->d_nsel, g->inst_selb);
}

// up to k paths per selected endpoint, in slots q * k + r
template <typename T>
void search_stage(tdp_graph g, int k, float slack_limit, hipStream_t s) {
  const T limit = (T)slack_limit;
  switch (g->side_k) {
    case 1: launch_search<T, 1>(g, k, limit, s); break;
    case 2: launch_search<T, 2>(g, k, limit, s); break;
    case 4: launch_search<T, 4>(g, k, limit, s); break;
    case 8: launch_search<T, 8>(g, k, limit, s); break;
    case 16: launch_search<T, 16>(g, k, limit, s); break;
    default: launch_search<T, 32>(g, k, limit, s); break;
  }
}

// the slots sorted by (instance, path slack), stable
template <typename T>
Sorted<uint64_t> slot_sort_stage(tdp_graph g, int k, hipStream_t s) {
  const int cap = g->slot_cap;
  hipLaunchKernelGGL(k_slot_keys<T>, dim3(std::min(1024, nb(cap, 256))), dim3(256), 0, s, g->topo, k, g->d_nsel,
                     g->sel_list, (const T *)g->slot_key, g->d_nslots, g->sort_k0, g->sort_v0);
  return radix_sort(g->sort_k0, g->sort_v0, g->sort_k1, g->sort_v1, cap, g->d_nslots,
                    sizeof(T) == 4 ? g->key_bits32 : 64, 11, g->sort_hist, s);
}

void ptr_tail(const int32_t *d_num_paths, const int32_t *len, int32_t *ptr, hipStream_t s) {
  hipLaunchKernelGGL(k_ptr_tail, dim3(1), dim3(1), 0, s, d_num_paths, len, ptr);
}

template <typename T>
void extract_impl(tdp_graph g, int n, int k, int K, float slack_limit, hipStream_t s) {
  const Topo &tp = g->topo;
  prof_begin(g, TDP_STAGE_SELECT, s);
  select_stage<T>(g, n, s);
  prof_end(g, TDP_STAGE_SELECT, s);
  prof_begin(g, TDP_STAGE_SEARCH, s);
  search_stage<T>(g, k, slack_limit, s);
  prof_end(g, TDP_STAGE_SEARCH, s);
  // ordering
  prof_begin(g, TDP_STAGE_ORDER, s);
  // the most slots the call can have: the endpoints selected times k
  const long long most = (n < 0 ? (long long)tp.E : std::min((long long)tp.E, (long long)n * tp.num_inst)) * k;
  int slot_bits = 1;
  while ((1ll << slot_bits) < most) ++slot_bits;
  if (sizeof(T) == 4 && most <= ORDER_ONE) {
    hipLaunchKernelGGL(k_order_one, dim3(1), dim3(1024), 0, s, tp, k, K, g->d_nsel, g->sel_list, g->inst_selb,
                       (const float *)g->slot_key, g->slot_len, g->d_nslots, g->out_slot, g->slot_out, g->path_ptr,
                       g->d_num_paths);
  } else if (sizeof(T) == 4 && g->key_bits32 + slot_bits <= 64) {
    const OrderBuf ob{g->sort_k0, g->sort_k1, g->order_hist, g->order_total, g->order_flags,
                      (int)std::min<long long>(LOOK_MAX, 4ll * g->spin_limit)};
    // (no more workgroups than it can have slots for: with more slots they leave)
    const long long ranked = std::min(most, (long long)tp.num_inst * RANK_MOST);
    hipLaunchKernelGGL(k_rank, dim3((int)std::min<long long>(1024, (ranked + 63) / 64)), dim3(1024), 0, s, tp, k,
                       slot_bits, g->d_nsel, g->sel_list, g->inst_selb, (const float *)g->slot_key, ob.w0, ob.flags + ORDER_GROUPS);
    hipLaunchKernelGGL(k_order, dim3((int)std::min<long long>(ORDER_GROUPS, (most + ORDER_RUN - 1) / ORDER_RUN)),
                       dim3(1024), 0, s, tp, k, K, g->key_bits32, slot_bits, g->d_nsel, g->sel_list, g->inst_selb,
                       (const float *)g->slot_key, g->slot_len, ob, g->d_nslots, g->out_slot, g->slot_out, g->path_ptr,
                       g->d_num_paths, g->d_err);
  } else {
    const Sorted<uint64_t> so = slot_sort_stage<T>(g, k, s);
    const Look lk{g->look_st, g->look_ctr, g->d_err};
    hipLaunchKernelGGL(k_path_out<T>, dim3(std::min(256, nb(g->slot_cap, OUT_TILE))), dim3(256), 0, s, k, K, lk,
                       g->d_nslots, g->inst_selb, so.keys, so.vals, g->slot_len, g->out_slot, g->slot_out, g->path_ptr,
                       g->d_num_paths);
  }
  prof_end(g, TDP_STAGE_ORDER, s);
  // walk
  prof_begin(g, TDP_STAGE_WALK, s);
  hipLaunchKernelGGL(k_walk<T>, dim3(nb(g->max_out, WALK_PATHS)), dim3(4 * WALK_PATHS), 0, s, tp, k, g->d_num_paths,
                     g->out_slot,
                     g->sel_list, g->slot_dev, g->slot_par, (const T *)g->slot_key, g->node, node_words<T>(g->side_k),
                     g->path_ptr, g->path_pins, g->path_int, g->path_ep, g->path_epi, g->path_rank,
                     (T *)g->path_slack, g->d_err, g->pin_cap, g->d_nslots);
  prof_end(g, TDP_STAGE_WALK, s);
}

template void extract_impl<float>(tdp_graph, int, int, int, float, hipStream_t);
template void extract_impl<double>(tdp_graph, int, int, int, float, hipStream_t);
template void select_stage<float>(tdp_graph, int, hipStream_t);
template void select_stage<double>(tdp_graph, int, hipStream_t);
template void search_stage<float>(tdp_graph, int, float, hipStream_t);
template void search_stage<double>(tdp_graph, int, float, hipStream_t);
template Sorted<uint64_t> slot_sort_stage<float>(tdp_graph, int, hipStream_t);
template Sorted<uint64_t> slot_sort_stage<double>(tdp_graph, int, hipStream_t);

}  // namespace tdp
