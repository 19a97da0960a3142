// Static timing analysis kernels (Sec. II-B, Eqs. 2-4; net delay Eq. 7).
//
// One update is:
//   net pass   every net as a segment of a 64-lane chunk (driver lane, then
//              its sinks): pin positions, the RC delay into each sink
//              (kappa * L^2 with L Manhattan, or the sink's Elmore delay),
//              the driver's load (star model, a segmented sum); start points
//              get arrival and transition.
//   forward    one lane per combinational input pin, a cell's inputs adjacent:
//              arrival = segmented max over inputs of (driver arrival + net
//              delay + table delay at the input's transition, under the Elmore
//              model the driver's degraded by the wire, and the output load),
//              output transition = segmented max of the table transitions, the
//              critical input = lowest lane attaining the max; the cell's head
//              lane writes the output.  Some lanes per cell then make its node
//              record: hops up the critical chain and, with deviation lists on,
//              the cell's own deviations merged into the critical driver's list.
//   endpoint   slack at every D pin; WNS / TNS / count per instance in a
//              fixed-order two-level reduction.
//   backward   from the top; one lane per net pin: required time of a driver =
//              segmented min over its sinks of (sink required time - net delay);
//              a cell's inputs' are its output's minus the arc delays.
// Either sweep runs in one launch on a resident grid, its waves waiting for the
// words they read (the dataflow sweeps below), or in one launch per level:
// incremental updates, deviation lists in double precision, required times with
// a net wider than a chunk, and wherever sweep_mode asks for it.
// Tables live in LDS for the forward sweep.  Nets with more than 63 sinks
// take a one-thread-per-net path.
#include "tdp_flow.h"
#include "tdp_impl.h"
#include "tdp_look.h"
#include "tdp_prims.h"
#include "tdp_wave.h"
#include "tdp_tree.h"

namespace tdp {

__device__ __forceinline__ uint64_t pack2(float lo, float hi) {
  return (uint64_t)__float_as_uint(lo) | ((uint64_t)__float_as_uint(hi) << 32);
}

// A driver's {arrival, transition} as published words.  All ones means "not yet":
// NaNs that came in with the positions may have that pattern, and get another.
__device__ __forceinline__ uint64_t flow_word(float a, float s) {
  const uint64_t w = pack2(a, s);
  return w != W_EMPTY ? w : pack2(__builtin_nanf(""), __builtin_nanf(""));
}
__device__ __forceinline__ uint64_t flow_word(double a) {
  const uint64_t w = (uint64_t)__double_as_longlong(a);
  return w != W_EMPTY ? w : (uint64_t)__double_as_longlong(__builtin_nan(""));
}

struct FlowInit {
  uint64_t *w = nullptr;
  void *r = nullptr;              // the backward sweep's published words and their count
  int nr = 0;
  int32_t *err = nullptr;  // cleared at the start of every update
  SweepShare *fw = nullptr, *bw = nullptr;  // of the sweeps whose words are reset: a new sweep each
  const uint32_t *tag = nullptr;  // the graph's pass counter and whether the last sweep gave up
  uint64_t *node = nullptr;
  uint32_t *cd = nullptr;
  int words = 0;                  // of a node record
  int seed = 1;  // 0: start points are never published (self-test of the bounded waits)
  int reset_blocks = 0;  // trailing workgroups of the net pass that reset the words
};

// Marks of an incremental arrival update (all null for a full one), as
// stamps: an entry equal to the update's epoch is set, any other value is
// not, so nothing is cleared between updates.  A chunk is re-timed when the
// net pass marked it or when a driver of one of its inputs changed in this
// update, which each of its lanes reads for itself (no pushing of marks
// along fanout lists).
struct IncFlags {
  int32_t epoch = 0;
  int32_t *arr = nullptr;               // [n_fw_chunks] the net pass changed an input's delay or the load
  int32_t *lst = nullptr;               // [n_fw_chunks] the chunk's arrivals were re-timed
  int32_t *drv_chg = nullptr;           // [M] the driver's arrival or transition changed
  int32_t *drv_lchg = nullptr;          // [M] its deviation list, hop records or chain depth changed
  const int32_t *snk_chunk = nullptr;   // [A] forward chunk of a combinational input
  const int32_t *nm = nullptr;          // [n_nm_chunks] the net chunk holds a moved cell's pin
};

template <typename T>
__device__ __forceinline__ bool same_bits(T a, T b) {
  if constexpr (sizeof(T) == 4) return __float_as_uint((float)a) == __float_as_uint((float)b);
  else return __double_as_longlong((double)a) == __double_as_longlong((double)b);
}

// v[0, n) = x, 16-byte stores where the alignment allows
__device__ __forceinline__ void fill_u32(uint32_t *p, size_t n, uint32_t x, size_t tid, size_t nth) {
  size_t h = ((16 - ((uintptr_t)p & 15)) & 15) / 4;
  h = h < n ? h : n;
  if (tid < h) p[tid] = x;
  uint4 *q = (uint4 *)(p + h);
  const size_t n4 = (n - h) / 4;
  const uint4 xx = make_uint4(x, x, x, x);
  for (size_t i = tid; i < n4; i += nth) q[i] = xx;
  const size_t t0 = h + n4 * 4;
  if (tid < n - t0) p[t0 + tid] = x;
}

// The words the dataflow sweeps poll return to "not yet published" at the
// start of every update (the start points' words are seeded by the net pass
// itself, so they are left out here): streaming stores in workgroups of their
// own beside the net pass's gathers.  The tagged words need this only after a
// sweep that gave up, which leaves some of them of an older pass.
template <typename T>
__device__ __forceinline__ void flow_reset(const FlowInit &fl, const Topo &tp, int b) {
  constexpr int N = sizeof(T) / 4;
  const size_t nth = (size_t)fl.reset_blocks * blockDim.x, tid = (size_t)b * blockDim.x + threadIdx.x;
  const size_t nc = (size_t)(tp.M - tp.n_start);
  if (tid == 0) {  // (here: at the head of the net pass its scalar loads cost every wave, 120 us against 116 at 1M cells)
    if (fl.fw) new_sweep(fl.fw);
    if (fl.bw) new_sweep(fl.bw);
  }
  if (fl.w) fill_u32((uint32_t *)(fl.w + (size_t)N * tp.n_start), 2 * N * nc, ~0u, tid, nth);
  if (fl.r) fill_u32((uint32_t *)fl.r, (size_t)fl.nr * N, ~0u, tid, nth);
  if (fl.w && fl.tag[1]) {
    // id 0 in both halves (a sweep that gives up again reads them as ids)
    // under the previous pass's tag, where a hop word or a list entry has it
    const uint32_t old = (fl.tag[0] - 1) << 30;
    for (size_t i = tid; i < nc * fl.words; i += nth)
      fl.node[i] = i % fl.words < HOP_WORDS ? (uint64_t)old : (uint64_t)old << 32;
    fill_u32(fl.cd + tp.n_start, nc, old, tid, nth);
  }
}

template <typename T>
__device__ __forceinline__ void start_point(const Topo &tp, const LutView &L, int v, T ld, T in_slew, T clk_slew,
                                            T *__restrict__ at, T *__restrict__ slew, V2<T> *__restrict__ as,
                                            uint32_t *__restrict__ cdep, const FlowInit &fl) {
  T a = 0, s = in_slew;
  if (v >= tp.n_pi && v < tp.n_start) lut_pair<T>(L, tp.ff_type[v - tp.n_pi], clk_slew, ld, a, s);
  if (v < tp.n_start) {
    at[v] = a;
    slew[v] = s;
    as[v] = v2<T>(a, s);
    // (an incremental pass, without a tag, leaves the depths as they are)
    if (fl.tag) cdep[v] = (fl.tag[0] - (fl.seed ? 0 : 1)) << 30;
    // seed the start points' words of the dataflow sweeps
    if (fl.w) {
      if constexpr (sizeof(T) == 4) {
        fl.w[v] = fl.seed ? flow_word(a, s) : W_EMPTY;
      } else {
        fl.w[2 * (size_t)v] = fl.seed ? flow_word(a) : W_EMPTY;
        fl.w[2 * (size_t)v + 1] = fl.seed ? flow_word(s) : W_EMPTY;
      }
    }
  }
}

// ------------------------------------------------------------- net pass
// one net chunk of the net pass (TREE: the spanning-tree model)
template <typename T, bool TREE>
__device__ __forceinline__ void netpass_chunk(const Topo &tp, const LutView &L, int chunk, const float2 *__restrict__ xy,
                                              const NetModel<T> &nm, T cw, T in_slew, T clk_slew,
                                              T *__restrict__ load, T *__restrict__ dnet, T *__restrict__ dnet_nm,
                                              float2 *__restrict__ cxy_nm, T *__restrict__ at, T *__restrict__ slew,
                                              V2<T> *__restrict__ as, uint32_t *__restrict__ cdep, const FlowInit &fl,
                                              const IncFlags &inc) {
  const int lane = wave_lane();
  const int k = chunk * CHUNK + lane;
  const int4 rec = tp.nm_rec[k];
  const int p = rec.x, cell = rec.y;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  // pin coordinate = cell coordinate + offset; differences are taken as
  // (cell - cell) + (offset - offset), exact to the rounding of the result
  // rather than of a die-scale sum.  A port has no cell and its offset is its
  // position: for the wire lengths it is taken as the base (offset 0), so a
  // port next to a cell far from the origin does not cancel two die-scale
  // numbers
  const float2 q = cell >= 0 ? xy[cell] : make_float2(0.f, 0.f);
  cxy_nm[k] = q;  // kept for the weighted-average wirelength at these positions
  const float fox = tp.nm_ox[k], foy = tp.nm_oy[k];
  const T cx = cell >= 0 ? (T)q.x : (T)fox, cy = cell >= 0 ? (T)q.y : (T)foy;
  const T ox = cell >= 0 ? (T)fox : (T)0, oy = cell >= 0 ? (T)foy : (T)0;
  const T cxd = __shfl(cx, head, 64), cyd = __shfl(cy, head, 64);
  const T oxd = __shfl(ox, head, 64), oyd = __shfl(oy, head, 64);
  const bool sink = p >= 0 && lane != head;
  T len, dn = 0;
  if constexpr (TREE) {
    const ChunkTree<T> tr = tree_chunk_build<T>(cw, lane, head, tail, sink, q.x, q.y, fox, foy, cx, cy, ox, oy,
                                                sink ? (T)tp.type_cap[(rec.w >> 16) & 255] : (T)0);
    len = tr.len;
    dn = tree_chunk_delay<T>(nm, tr);
  } else {
    len = sink ? fabs((cxd - cx) + (oxd - ox)) + fabs((cyd - cy) + (oyd - oy)) : (T)0;
  }
  if (sink) {
    if constexpr (!TREE) dn = nm.delay(len, nm.elmore ? (T)tp.type_cap[(rec.w >> 16) & 255] : (T)0);
    dnet[p - tp.M] = dn;
    dnet_nm[k] = dn;
    // incremental: every sink of a re-timed net gets its chunk re-timed
    if (inc.arr && p - tp.M < tp.A) inc.arr[inc.snk_chunk[p - tp.M]] = inc.epoch;
  }
  const T wl = seg_sum(len, lane, head, tail);
  if (p >= 0 && lane == head) {
    const T ld = (T)tp.net_cpin[p] + cw * wl;
    load[p] = ld;
    start_point<T>(tp, L, p, ld, in_slew, clk_slew, at, slew, as, cdep, fl);
    // incremental: a combinational driver's cell sees its new load
    if (inc.arr && p >= tp.n_start) inc.arr[inc.snk_chunk[tp.comb_inptr[p - tp.n_start]]] = inc.epoch;
  }
}

template <typename T, bool TREE>
__global__ void __launch_bounds__(256) k_netpass(Topo tp, LutView L, const float2 *__restrict__ xy, NetModel<T> nm,
                                                  T cw, T in_slew,
                                                  T clk_slew, T *__restrict__ load, T *__restrict__ dnet,
                                                  T *__restrict__ dnet_nm, float2 *__restrict__ cxy_nm,
                                                  T *__restrict__ at, T *__restrict__ slew,
                                                  V2<T> *__restrict__ as, uint32_t *__restrict__ cdep, FlowInit fl) {
  if (blockIdx.x == 0 && threadIdx.x == 0 && fl.err) *fl.err = 0;
  const int main_blocks = (int)gridDim.x - fl.reset_blocks;
  if ((int)blockIdx.x >= main_blocks) {
    flow_reset<T>(fl, tp, (int)blockIdx.x - main_blocks);
    return;
  }
  const int chunk = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= tp.n_nm_chunks) return;
  netpass_chunk<T, TREE>(tp, L, chunk, xy, nm, cw, in_slew, clk_slew, load, dnet, dnet_nm, cxy_nm, at, slew, as,
                         cdep, fl, IncFlags{});
}

// the net pass over the marked net chunks of an incremental update (the same
// computation per chunk, so the results are those of a full pass)
template <typename T, bool TREE>
__global__ void __launch_bounds__(256) k_netpass_marked(Topo tp, LutView L, const float2 *__restrict__ xy,
                                                         NetModel<T> nm, T cw, T in_slew, T clk_slew,
                                                         T *__restrict__ load, T *__restrict__ dnet,
                                                         T *__restrict__ dnet_nm, float2 *__restrict__ cxy_nm,
                                                         T *__restrict__ at, T *__restrict__ slew,
                                                         V2<T> *__restrict__ as, uint32_t *__restrict__ cdep,
                                                         IncFlags inc) {
  const int chunk = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= tp.n_nm_chunks || inc.nm[chunk] != inc.epoch) return;
  netpass_chunk<T, TREE>(tp, L, chunk, xy, nm, cw, in_slew, clk_slew, load, dnet, dnet_nm, cxy_nm, at, slew, as,
                         cdep, FlowInit{}, inc);
}

// nets too wide for one chunk: one thread per net (tree_wl: the spanning-tree
// model, whose delays the tree kernel wrote)
template <typename T>
__global__ void k_netpass_big(Topo tp, LutView L, const float *__restrict__ x, const float *__restrict__ y, NetModel<T> nm,
                              const T *__restrict__ tree_wl, T cw, T in_slew, T clk_slew, T *__restrict__ load,
                              T *__restrict__ dnet,
                              T *__restrict__ at, T *__restrict__ slew, V2<T> *__restrict__ as,
                              uint32_t *__restrict__ cdep, FlowInit fl) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= tp.n_big) return;
  const int v = tp.big_net[i];
  const int dc = tp.drv_cell[v];
  // a port driver: its position as the base (see the chunk form)
  const T cx = dc >= 0 ? (T)x[dc] : (T)tp.drv_ox[v], cy = dc >= 0 ? (T)y[dc] : (T)tp.drv_oy[v];
  const T ox = dc >= 0 ? (T)tp.drv_ox[v] : (T)0, oy = dc >= 0 ? (T)tp.drv_oy[v] : (T)0;
  T wl = tree_wl ? tree_wl[v] : (T)0;
  for (int k = tp.net_ptr[v]; !tree_wl && k < tp.net_ptr[v + 1]; ++k) {
    const int t = tp.net_sink[k];
    const int sc = tp.snk_cell[t];
    const T len = fabs((cx - (T)x[sc]) + (ox - (T)tp.snk_ox[t])) + fabs((cy - (T)y[sc]) + (oy - (T)tp.snk_oy[t]));
    dnet[t] = nm.delay(len, nm.elmore ? (T)tp.snk_cap[t] : (T)0);
    wl += len;
  }
  const T ld = (T)tp.net_cpin[v] + cw * wl;
  load[v] = ld;
  start_point<T>(tp, L, v, ld, in_slew, clk_slew, at, slew, as, cdep, fl);
}

// -------------------------------------------------------------- forward
// One launch per level l does two jobs in separate workgroups: the arrivals
// of level l (the first n_arr workgroups) and, one level behind, the chain
// depths and deviation lists of level l-1, whose critical inputs the previous
// launch settled.  A cell's list extends its critical input's driver's list,
// a dependent load; running it beside the next level's arrivals keeps that
// round trip off the arrival chain.  fw_a keeps each input's arrival through
// its arc (by input) for the list job.
// a cell's maximum arrival, worst transition and the lane of its first input
// attaining the maximum (the head when none does, e.g. NaN), from its inputs'
// a and o; w: the lane's record's last word
template <typename T>
__device__ __forceinline__ void cell_max(T a, T o, bool valid, int w, int lane, T &best, T &so, int &argl) {
  const int head = w & 63, tail = (w >> 8) & 63;
  if (((w >> 24) & 127) <= 4) {  // every cell of the chunk has <= 4 inputs
    T ua[4], uo[4];
    seg_fetch<4>(a, head, tail, ua);
    seg_fetch<4>(o, head, tail, uo);
    int aj, oj;
    best = max_first<4>(ua, aj);
    so = max_first<4>(uo, oj);
    argl = head + aj;
  } else {
    best = seg_max(a, lane, head, tail);
    so = seg_max(o, lane, head, tail);
    const int arg0 = seg_min((valid && a == best) ? lane : 64, lane, head, tail);
    argl = arg0 <= tail ? arg0 : head;
  }
}

template <typename T>
__device__ __forceinline__ void fw_arrivals(const Topo &tp, const LutView &L, float *s_lut, int chunk, int ch1,
                                            const T *__restrict__ load, const T *__restrict__ dnet,
                                            T *__restrict__ at, T *__restrict__ slew, V2<T> *__restrict__ as,
                                            T *__restrict__ darc, int32_t *__restrict__ crit, T *__restrict__ fw_a,
                                            uint64_t *__restrict__ node, int words, uint32_t tag,
                                            const IncFlags &inc) {
  const int lane = wave_lane();
  // the record and the inputs' loads are issued before the tables are
  // staged, so the latencies overlap (a wave past the level's last chunk
  // reads that chunk's records again and then leaves)
  const int4 rec = tp.fw_rec[(chunk < ch1 ? chunk : ch1 - 1) * CHUNK + lane];
  const int2 ex = tp.fw_ext[(chunk < ch1 ? chunk : ch1 - 1) * CHUNK + lane];
  const int t = rec.x, s = rec.y, c = rec.z;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  const bool valid = t >= 0 && chunk < ch1;
  T ld = 0, dn = 0;
  V2<T> w = v2<T>(0, 0), old = v2<T>(0, 0);
  if (valid) {
    ld = load[tp.n_start + c];
    w = as[s];
    dn = dnet[t];
  }
  // incremental: whether the net pass marked the chunk or an input's driver
  // changed, and the cell's previous output and hop (issued with the same loads)
  ulonglong2 old_hop = make_ulonglong2(0, 0);
  bool mark = false;
  if (inc.arr && valid) {
    mark = inc.drv_chg[s] == inc.epoch || inc.arr[chunk] == inc.epoch;
    if (lane == head) {
      old = as[tp.n_start + c];
      old_hop = *reinterpret_cast<const ulonglong2 *>(node + (size_t)c * words);
    }
  }
  stage_lut(L, s_lut);
  if (chunk >= ch1) return;
  if (inc.arr) {  // only marked chunks, whose cells' lists follow
    if (__ballot(mark) == 0) return;
    if (lane == 0) inc.lst[chunk] = inc.epoch;
  }
  T a = -pos_inf<T>(), o = 0;
  if (valid) {
    const T a_in = w.x + dn;
    T d;
    lut_lds<T>(s_lut, L.nt, L.ns, L.nl, (rec.w >> 16) & 255, sink_slew<T>(L.net_model, w.y, dn), ld, d, o);
    at[tp.M + t] = a_in;
    darc[t] = d;
    a = a_in + d;
    fw_a[t] = a;  // for the list job
  }
  T best, so;
  int argl;
  cell_max<T>(a, o, valid, rec.w, lane, best, so, argl);
  const uint64_t h0 = pack_ids(__shfl(t, argl & 63, 64), __shfl(s, argl & 63, 64), tag);
  const uint64_t h1 = pack_ids(__shfl(ex.x, argl & 63, 64), __shfl(ex.y, argl & 63, 64), tag);
  if (valid && lane == head) {
    const int v = tp.n_start + c;
    if (inc.arr && (!same_bits(old.x, best) || !same_bits(old.y, so)))
      inc.drv_chg[v] = inc.epoch;  // a changed output re-times the cells it drives
    at[v] = best;
    slew[v] = so;
    as[v] = v2<T>(best, so);
    crit[c] = argl - head;
    // (the records above copy this hop; the tag is the last full pass's)
    if (inc.arr && (old_hop.x != h0 || old_hop.y != h1)) inc.drv_lchg[v] = inc.epoch;
    *reinterpret_cast<ulonglong2 *>(node + (size_t)c * words) = make_ulonglong2(h0, h1);
  }
}

// Lists of cells [.., lc1), LG lanes per cell: the rest of a cell's node
// record (the arrival job wrote its own hop): the first three hops of its
// critical input's driver, its chain depth, and its deviation list: the
// driver's list merged with the cell's own deviations.  Lane j holds entry j
// of the driver's list and deviation j of the cell; every value's place in the
// merged list is its rank (own deviations in front of equal entries, in arc
// order among themselves), counted from broadcasts and ballots, and is stored
// there directly.  Two dependent loads (the own hop, then everything else) and
// a few dozen instructions, whatever KM; one lane inserting into a list in
// registers took a chain of several hundred at KM = 16.
// ranks of a group's values in the merged list: `shift` own deviations go in
// front of lane j's entry e, and lane j's own deviation d (index i0 of the
// cell's inputs, +inf for none) goes to `rank`.  dev(i) gives every lane of
// the group the cell's deviation i (+inf for the critical input and past the
// last one), i < nmax; `base`: the group's first lane, `group`: its lanes.
template <typename T, class F>
__device__ __forceinline__ void list_ranks(T e, T d, int i0, int nmax, unsigned long long group, F &&dev, int &shift,
                                           int &rank) {
  shift = 0;
  rank = 0;
  for (int i = 0; i < nmax; ++i) {
    const T di = dev(i);
    const bool own = di < pos_inf<T>();
    shift += own && di <= e;
    const int less = __popcll(__ballot(e < di) & group);
    rank += i == i0 ? less : (own && (di < d || (di == d && i < i0)));
  }
}

// Cells with more inputs than a group has lanes: the deviations of the inputs from
// the LG-th on go into the driver's list first, LG at a time and the last ones
// first (equal ones of inputs before them then go in front), and the cell's first
// LG inputs follow as they do for other cells.  e: lane j's entry of the list;
// best: the cell's arrival; arc(i): the arrival through arc i < n of the group's
// cell, all lanes' at once, whether the wave is to go on with it in `go`.  The new
// list passes through LDS.  With deviations one by one from memory, once for every LG
// of them, the update of 100,000 cells of up to 20 inputs took 1,150 us (k = 2 or 8),
// with this 396.
template <typename T, int KM, class F>
__device__ __forceinline__ Dev<T> absorb_wide(Dev<T> e, T best, int n, int nmax, int arg, int t0,
                                              unsigned long long group, bool &go, F &&arc) {
  constexpr int LG = list_lanes(KM);
  __shared__ T s_cost[256];
  __shared__ int32_t s_sink[256];
  const int lane = wave_lane(), j = lane & (LG - 1), base = lane & ~(LG - 1);
  const int first = (int)threadIdx.x - j;  // the group's part of the arrays
  for (int b = (nmax - 1) / LG * LG; b >= LG; b -= LG) {
    const int i = b + j;
    const T a = arc(i);
    if (!go) break;
    const T d = i < n && i != arg && best - a < pos_inf<T>() ? best - a : pos_inf<T>();
    int shift, rank;
    list_ranks(e.cost, d, j, min(LG, nmax - b), group, [&](int q) { return __shfl(d, base + q, 64); }, shift, rank);
    if (d < pos_inf<T>() && rank < KM) {
      s_cost[first + rank] = d;
      s_sink[first + rank] = t0 + i;
    }
    if (j < KM && j + shift < KM) {
      s_cost[first + j + shift] = e.cost;
      s_sink[first + j + shift] = e.sink;
    }
    wave_lds_sync();
    if (j < KM) e = Dev<T>{s_cost[first + j], s_sink[first + j]};
    wave_lds_sync();
  }
  return e;
}

template <typename T, int KM>
__device__ __forceinline__ void fw_lists(const Topo &tp, int c, int lc1, const T *__restrict__ at,
                                         const T *__restrict__ fw_a, uint32_t *__restrict__ cdep,
                                         uint64_t *__restrict__ node, uint32_t tag, const IncFlags &inc) {
  constexpr int LG = list_lanes(KM), W = node_words<T>(KM);
  const int lane = wave_lane(), j = lane & (LG - 1), base = lane & ~(LG - 1);
  bool live = c < lc1;
  const int cc = live ? c : lc1 - 1;  // (spare groups read the last cell's record and store nothing)
  const uint64_t own = node[(size_t)cc * W];
  const int t0 = tp.comb_inptr[cc], n = tp.comb_inptr[cc + 1] - t0;
  const int pred = (int)(uint32_t)(own >> 32), arg = id30((uint32_t)own) - t0;
  if (inc.lst) {  // incremental: the cell was re-timed or its critical driver's record changed
    const bool mark = inc.drv_lchg[pred] == inc.epoch || inc.lst[inc.snk_chunk[t0]] == inc.epoch;
    live = live && mark;
  }
  const bool chain = pred >= tp.n_start;
  const int pc = chain ? pred - tp.n_start : 0;
  const T best = at[tp.n_start + cc];
  const uint32_t cd = ((cdep[pred] + 1) & ID_MASK) | tag << 30;
  const T a0 = j < n ? fw_a[t0 + j] : pos_inf<T>();
  uint64_t hw = j & 1 ? pack_ids(0, 0, tag) : pack_ids(-1, -1, tag);
  if (chain && j < HOP_WORDS - 2) hw = node[(size_t)pc * W + j];
  Dev<T> e{pos_inf<T>(), -1};
  if constexpr (KM > 1) {
    if (chain && j < KM) e = list_entry<T, KM>(node, pc, j);
  }
  bool changed = false;
  if (inc.lst) {
    if (live && j < HOP_WORDS - 2) changed = node[(size_t)cc * W + 2 + j] != hw;
    if (live && j == 0) changed = changed || cdep[tp.n_start + cc] != cd;
  }
  if (live && j < HOP_WORDS - 2) node[(size_t)cc * W + 2 + j] = hw;
  if (live && j == 0) cdep[tp.n_start + cc] = cd;
  const unsigned long long group = ((1ull << LG) - 1) << base;
  if constexpr (KM > 1) {
    auto place = [&](int pos, Dev<T> v) {
      if (!live || pos >= KM) return;
      if (inc.lst) {
        const Dev<T> o = list_entry<T, KM>(node, cc, pos);
        changed = changed || !same_bits(o.cost, v.cost) || o.sink != v.sink;
      }
      store_entry<T, KM>(node, cc, pos, v, tag);
    };
    const int nmax = wave_max_int(n);
    if (nmax > LG) {
      bool go = true;
      e = absorb_wide<T, KM>(e, best, n, nmax, arg, t0, group, go, [&](int i) { return i < n ? fw_a[t0 + i] : pos_inf<T>(); });
    }
    int shift, rank;
    const T d = j < n && j != arg ? best - a0 : pos_inf<T>();
    list_ranks(e.cost, d, j, min(nmax, LG), group, [&](int i) { return __shfl(d, base + i, 64); }, shift, rank);
    if (d < pos_inf<T>()) place(rank, Dev<T>{d, t0 + j});
    if (j < KM) place(j + shift, e);
  }
  if (inc.lst) {
    const unsigned long long any = __ballot(changed);
    // the cells this one drives may take it as their critical input
    if (live && j == 0 && (any & group)) inc.drv_lchg[tp.n_start + cc] = inc.epoch;
  }
}

// arrival chunks [ch0, ch1) in workgroups [0, n_arr); lists of cells [lc0, lc1)
// in the rest
template <typename T, int KM>
__global__ void __launch_bounds__(256) k_forward(Topo tp, LutView L, int ch0, int ch1, int n_arr, int lc0, int lc1,
                                                  const T *__restrict__ load, const T *__restrict__ dnet,
                                                  T *__restrict__ at, T *__restrict__ slew, V2<T> *__restrict__ as,
                                                  T *__restrict__ darc, int32_t *__restrict__ crit,
                                                  uint32_t *__restrict__ cdep, uint64_t *__restrict__ node,
                                                  T *__restrict__ fw_a, const uint32_t *__restrict__ d_tag,
                                                  IncFlags inc) {
  extern __shared__ float4 s_lut4[];
  float *s_lut = (float *)s_lut4;
  const int wave = threadIdx.x >> 6;
  const uint32_t tag = *d_tag & 3u;
  if ((int)blockIdx.x < n_arr)
    fw_arrivals<T>(tp, L, s_lut, ch0 + blockIdx.x * 4 + wave, ch1, load, dnet, at, slew, as, darc, crit, fw_a, node,
                   node_words<T>(KM), tag, inc);
  else
    fw_lists<T, KM>(tp, lc0 + ((blockIdx.x - n_arr) * 256 + threadIdx.x) / list_lanes(KM), lc1, at, fw_a, cdep, node,
                    tag, inc);
}

// ------------------------------------------------------------- endpoints
// Slack at every D pin (SLACK; otherwise ep_slack holds them already), and per
// instance {min, sum of negatives, count of negatives}: a workgroup takes one part
// of an instance's endpoints (job: the instance, its number of parts, this one),
// and the last workgroup of the instance to be done folds its parts, in order.
// One launch: 9 us at 20,000 endpoints, 13 at 240,000; as three (slacks, partial
// sums, one thread's fold) 17 and 23.  Every instance counts its own workgroups
// and has no more of them than its own endpoints ask for: with one count, one
// number of parts and one fold for all, the update of 1,000 designs of 100 cells
// took 1,070 us, with this 64 (4,000 of 60: 4,111 and 82; 24 of 3,000: 91 and 66).
template <typename T, bool SLACK>
__global__ void __launch_bounds__(256) k_endpoint(Topo tp, const int32_t *__restrict__ ep_base,
                                                   const int4 *__restrict__ jobs,
                                                   const double *__restrict__ inst_req, const T *__restrict__ dnet,
                                                   T *__restrict__ at, T *__restrict__ rat, T *__restrict__ ep_slack,
                                                   double *__restrict__ part, uint32_t *__restrict__ counts,
                                                   double *__restrict__ summary) {
  __shared__ double smin[256], ssum[256], scnt[256];
  __shared__ int s_last;
  const int4 job = jobs[blockIdx.x];
  const int inst = job.x, parts = job.y, j = job.z;
  const int b = ep_base[inst], e = ep_base[inst + 1];
  const int len = e - b;
  const int lo = b + (int)((long long)len * j / parts), hi = b + (int)((long long)len * (j + 1) / parts);
  const T req = SLACK ? (T)inst_req[inst] : (T)0;
  double mn = 0.0, sm = 0.0, ct = 0.0;
  for (int f = lo + threadIdx.x; f < hi; f += blockDim.x) {
    T sl;
    if constexpr (SLACK) {
      const int t = tp.A + f;
      const T a = at[tp.snk_drv[t]] + dnet[t];
      sl = req - a;
      at[tp.M + t] = a;
      rat[tp.M + t] = req;
      ep_slack[f] = sl;
    } else {
      sl = ep_slack[f];
    }
    const double s = (double)sl;
    if (s < 0) {
      mn = s < mn ? s : mn;
      sm += s;
      ct += 1.0;
    }
  }
  auto fold = [&]() {
    smin[threadIdx.x] = mn;
    ssum[threadIdx.x] = sm;
    scnt[threadIdx.x] = ct;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if ((int)threadIdx.x < o) {
        smin[threadIdx.x] = fmin(smin[threadIdx.x], smin[threadIdx.x + o]);
        ssum[threadIdx.x] += ssum[threadIdx.x + o];
        scnt[threadIdx.x] += scnt[threadIdx.x + o];
      }
      __syncthreads();
    }
  };
  fold();
  if (parts > 1) {
    if (threadIdx.x == 0) {
      pub_st(part + 3 * blockIdx.x + 0, smin[0]);
      pub_st(part + 3 * blockIdx.x + 1, ssum[0]);
      pub_st(part + 3 * blockIdx.x + 2, scnt[0]);
      stores_arrived();
      s_last = atomicAdd(counts + inst, 1u) == (uint32_t)parts - 1;
      if (s_last) pub_st(counts + inst, 0u);
    }
    __syncthreads();
    if (!s_last) return;
    mn = sm = ct = 0.0;
    if ((int)threadIdx.x < parts) {  // (at most 256)
      const double *p = part + 3 * ((size_t)blockIdx.x - j + threadIdx.x);
      mn = pub_ld(p);
      sm = pub_ld(p + 1);
      ct = pub_ld(p + 2);
    }
    fold();
  }
  if (threadIdx.x == 0) {
    summary[4 * inst + 0] = smin[0];
    summary[4 * inst + 1] = ssum[0];
    summary[4 * inst + 2] = scnt[0];
    summary[4 * inst + 3] = 0.0;
  }
}

// ------------------------------------------------------------- backward
// A net's pass gives each of its sinks its required time (a combinational
// input: its cell output's minus the arc delay; a flip-flop D pin: set at the
// endpoint), then its driver the minimum over the sinks of (sink required
// time - net delay).  Slack is rat - at, formed where it is exported.  The
// net delays are read in chunk-slot order (dnet_nm).
template <typename T>
__device__ __forceinline__ T sink_required(int p, T r_out, T da, T *__restrict__ rat) {
  const T ri = r_out != pos_inf<T>() ? r_out - da : pos_inf<T>();
  rat[p] = ri;
  return ri;
}

template <typename T>
__global__ void __launch_bounds__(256) k_backward(Topo tp, int ch0, int ch1, const T *__restrict__ dnet_nm,
                                                   const T *__restrict__ darc, T *__restrict__ rat) {
  const int lane = wave_lane();
  const int chunk = ch0 + blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= ch1) return;
  const int k = chunk * CHUNK + lane;
  const int4 rec = tp.nm_rec[k];
  const int p = rec.x, vo = rec.z;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  T r = pos_inf<T>();
  if (p >= 0 && lane != head) {
    const T dn = dnet_nm[k];
    const T rt = vo >= 0 ? sink_required<T>(p, rat[vo], darc[p - tp.M], rat) : rat[p];
    if (rt != pos_inf<T>()) r = rt - dn;
  }
  r = seg_min(r, lane, head, tail);
  if (p >= 0 && lane == head) rat[p] = r;
}

template <typename T>
__global__ void k_backward_big(Topo tp, int i0, int i1, const T *__restrict__ dnet, const T *__restrict__ darc,
                               T *__restrict__ rat) {
  const int i = i0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= i1) return;
  const int v = tp.big_net[i];
  T r = pos_inf<T>();
  for (int k = tp.net_ptr[v]; k < tp.net_ptr[v + 1]; ++k) {
    const int t = tp.net_sink[k];
    const int p = tp.M + t;
    const T rt = t < tp.A ? sink_required<T>(p, rat[tp.n_start + tp.snk_comb[t]], darc[t], rat) : rat[p];
    if (rt == pos_inf<T>()) continue;
    const T q = rt - dnet[t];
    r = q < r ? q : r;
  }
  rat[v] = r;
}

// ------------------------------------------------------ dataflow sweeps
// One launch per sweep on a resident grid: every workgroup of the launch is
// on the GPU at once (the grid is sized from the occupancy of the kernel, at
// most a few workgroups per compute unit), and wave w of the W waves owns
// chunks w, w + W, w + 2W, ... in dependency order (forward: level order;
// backward: reverse level order).  For each chunk a wave loads its static
// data (the next chunk's record is already in flight), waits until the words
// it reads are published, computes exactly what the per-level kernels
// compute, and publishes its own words.  A chunk waits only on chunks with
// smaller indices, and every wave takes its chunks in increasing order, so
// the smallest unfinished chunk always has its inputs and its owner at it:
// the sweep completes.  Where other streams' kernels keep workgroups out for
// long, those inside leave their fixed shares and take chunks by tickets
// (tdp_flow.h): the sweep completes whichever workgroups are inside.  The
// tables are staged in LDS once per workgroup, not once per chunk.
// Every wait is also bounded, so a broken assumption ends in a reported
// error, not a hang.  One lane per wave polls (the word its chunk is likely
// to see published last) before the others load theirs, which keeps the
// polling traffic of the waiting waves off the frontier's way.
//
// Forward.  Two kinds of workgroups share the launch.  Arrival waves take the
// chunks: a lane loads its driver's {arrival, transition} word, waiting only if
// it is not out yet; the cell's head lane publishes the output's word before
// anything else, then its cell's own hop, and with deviation lists every lane
// its input's arrival through its arc.  List waves take the cells in order,
// list_lanes lanes per cell as in the per-level list job: they wait for the
// cell's own hop (its arrival is out), then for the record of its critical
// input's driver, and publish the rest of the cell's record.  Every record word
// says by its tag whether it is this pass's, so each is waited for by itself
// and no fence is needed.  Arrivals never wait for lists, so the arrival chain
// runs at its own pace and the list chain trails it; in one wave that did
// both (lists of a chunk after the arrivals of its next) each level took the
// time of the slower of the two (200k cells, k = 10: 517 us against 149).
// Both kinds wait only on lower-numbered chunks or cells and take theirs in
// increasing order, so the lowest one not yet done can always run.
//
// An arrival through an arc, as the arrival waves publish it for the list
// waves, with the whole number of its pass: passes by level do not write these
// words, so any number of passes may lie between two that do.
__device__ __forceinline__ uint64_t pack_arc(float a, uint32_t pass) {
  return (uint64_t)__float_as_uint(a) | (uint64_t)pass << 32;
}
__device__ __forceinline__ uint32_t arc_pass(uint64_t w) { return (uint32_t)(w >> 32); }
__device__ __forceinline__ float arc_arrival(uint64_t w) { return __uint_as_float((uint32_t)w); }

// Words idx * N .. idx * N + N - 1 of every lane that wants them.  If some are
// not out yet, one lane first polls the last word of the highest-numbered
// missing driver (likely to be published last), so that a waiting wave polls
// one address rather than 64; then all missing words are loaded again
// together, one round trip per poll.  Bounded and left as load_or_wait.
template <int N, bool TICKETS>
__device__ __forceinline__ bool load_words(const uint64_t *base, int idx, bool want, uint64_t (&w)[N],
                                           const Waits<SWEEP_FORWARD> &wt) {
  bool miss = false;
#pragma unroll
  for (int q = 0; q < N; ++q) {
    w[q] = want ? pub_ld(base + (size_t)idx * N + q) : 0ull;
    miss = miss || w[q] == W_EMPTY;
  }
  if (!__ballot(miss)) return true;
  Polls<TICKETS, SWEEP_FORWARD> polls(wt);
  const uint64_t *const last = base + (size_t)wave_max_int(miss ? idx : -1) * N + N - 1;
  const bool first = wave_lane() == 0;
  uint64_t r;
  do {
    do r = first ? pub_ld(last) : 0ull;
    while (polls.missing(r == W_EMPTY));
    do {
      if (miss) {
        miss = false;
#pragma unroll
        for (int q = 0; q < N; ++q) {
          if (w[q] == W_EMPTY) w[q] = pub_ld(base + (size_t)idx * N + q);
          miss = miss || w[q] == W_EMPTY;
        }
      }
    } while (polls.missing(miss, false));
  } while (polls.resume(miss));
  return !polls.leave;
}

// A chunk's arrivals from its drivers' words, published and stored
template <typename T, int N>
__device__ __forceinline__ void arrive(const Topo &tp, const LutView &L, const float *s_lut, int4 rec, int2 ex, T ld, T dn,
                                       const uint64_t (&w)[N], T *__restrict__ at, T *__restrict__ slew,
                                       T *__restrict__ darc, int32_t *__restrict__ crit, uint64_t *__restrict__ node,
                                       int words, uint64_t *__restrict__ fa, uint64_t *__restrict__ fw,
                                       uint32_t pass) {
  const int lane = wave_lane();
  const uint32_t tag = pass & 3u;
  const int t = rec.x, s = rec.y, c = rec.z, ty = (rec.w >> 16) & 255;
  const int head = rec.w & 63;
  const bool valid = t >= 0;
  T a = -pos_inf<T>(), o = 0, a_in = 0, d = 0;
  if (valid) {
    T wa, ws;
    if constexpr (N == 1) {
      wa = __uint_as_float((uint32_t)w[0]);
      ws = __uint_as_float((uint32_t)(w[0] >> 32));
    } else {
      wa = __longlong_as_double((long long)w[0]);
      ws = __longlong_as_double((long long)w[N - 1]);
    }
    a_in = wa + dn;
    lut_lds<T>(s_lut, L.nt, L.ns, L.nl, ty, sink_slew<T>(L.net_model, ws, dn), ld, d, o);
    a = a_in + d;
  }
  T best, so;
  int argl;
  cell_max<T>(a, o, valid, rec.w, lane, best, so, argl);
  const bool is_head = valid && lane == head;
  const int v = tp.n_start + c;
  if (is_head) {
    if constexpr (N == 1) {
      pub_st(&fw[v], flow_word(best, so));
    } else {
      pub_st(&fw[2 * (size_t)v], flow_word(best));
      pub_st(&fw[2 * (size_t)v + 1], flow_word(so));
    }
  }
  const uint64_t h0 = pack_ids(__shfl(t, argl & 63, 64), __shfl(s, argl & 63, 64), tag);
  const uint64_t h1 = pack_ids(__shfl(ex.x, argl & 63, 64), __shfl(ex.y, argl & 63, 64), tag);
  if constexpr (N == 1) {
    if (fa && valid) pub_st(&fa[t], pack_arc(a, pass));
  }
  if (is_head) {
    pub_st(node + (size_t)c * words, h0);
    pub_st(node + (size_t)c * words + 1, h1);
    at[v] = best;
    slew[v] = so;
    crit[c] = argl - head;
  }
  if (valid) {
    at[tp.M + t] = a_in;
    darc[t] = d;
  }
}

// arrivals of chunks w0, w0 + W, ..., or (TICKETS) of those that tickets give;
// false if the wave left its share
template <typename T, bool TICKETS>
__device__ __forceinline__ bool flow_arrivals(const Topo &tp, const LutView &L, float *s_lut, int w0, int W,
                                              const T *__restrict__ load, const T *__restrict__ dnet,
                                              T *__restrict__ at, T *__restrict__ slew, T *__restrict__ darc,
                                              int32_t *__restrict__ crit, uint64_t *__restrict__ node, int words,
                                              uint64_t *__restrict__ fa, uint64_t *__restrict__ fw, uint32_t pass,
                                              const Waits<SWEEP_FORWARD> &wt) {
  constexpr int N = sizeof(T) / 4;  // words of a driver's {arrival, transition}
  const int lane = wave_lane();
  const int nch = tp.n_fw_chunks;
  uint64_t w[N];
  if constexpr (TICKETS) {
    stage_lut(L, s_lut);
    for (int chunk; (chunk = take_ticket(&wt.share()->ticket[0])) < nch;) {
      const int4 rec = tp.fw_rec[chunk * CHUNK + lane];
      const int2 ex = tp.fw_ext[chunk * CHUNK + lane];
      const bool valid = rec.x >= 0;
      const T ld = valid ? load[tp.n_start + rec.z] : (T)0, dn = valid ? dnet[rec.x] : (T)0;
      load_words<N, true>(fw, rec.y, valid, w, wt);
      arrive<T, N>(tp, L, s_lut, rec, ex, ld, dn, w, at, slew, darc, crit, node, words, fa, fw, pass);
    }
    return true;
  }
  int chunk = w0;
  const int4 norec = make_int4(-1, 0, 0, 0);
  int4 rec1 = norec, rec2 = norec;  // records of this wave's next two chunks
  int2 ex1 = make_int2(0, 0);
  T ld1 = 0, dn1 = 0;
  if (chunk < nch) {
    rec1 = tp.fw_rec[chunk * CHUNK + lane];
    ex1 = tp.fw_ext[chunk * CHUNK + lane];
  }
  if (chunk + W < nch) rec2 = tp.fw_rec[(chunk + W) * CHUNK + lane];
  stage_lut(L, s_lut);
  if (rec1.x >= 0) {
    ld1 = load[tp.n_start + rec1.z];
    dn1 = dnet[rec1.x];
  }
  for (; chunk < nch; chunk += W) {
    const int4 rec = rec1;
    const int2 ex = ex1;
    const T ld = ld1, dn = dn1;
    if (!load_words<N, false>(fw, rec.y, rec.x >= 0, w, wt)) return false;
    // the next chunks' static data, in flight behind this one
    rec1 = rec2;
    rec2 = norec;
    if (rec1.x >= 0) {
      ld1 = load[tp.n_start + rec1.z];
      dn1 = dnet[rec1.x];
    }
    if (chunk + W < nch) ex1 = tp.fw_ext[(chunk + W) * CHUNK + lane];
    if (chunk + 2 * W < nch) rec2 = tp.fw_rec[(chunk + 2 * W) * CHUNK + lane];
    arrive<T, N>(tp, L, s_lut, rec, ex, ld, dn, w, at, slew, darc, crit, node, words, fa, fw, pass);
  }
  return true;
}

// One turn of a wave's groups: the node record of cell c (c of the turn's cells
// that share the wave; spare groups repeat the last, last_c, with `on` false, and
// store nothing), whose inputs are the n from t0 on.  False if the wave left its
// share.
template <typename T, int KM, bool TICKETS>
__device__ __forceinline__ bool list_turn_of(const Topo &tp, int c, bool on, int last_c, int t0, int n,
                                             uint32_t *__restrict__ cdep, uint64_t *__restrict__ node,
                                             const uint64_t *__restrict__ fa, uint32_t pass, const Waits<SWEEP_FORWARD> &wt) {
  constexpr int LG = list_lanes(KM), NW = node_words<T>(KM);
  const uint32_t tag = pass & 3u;
  const int lane = wave_lane(), j = lane & (LG - 1), base = lane & ~(LG - 1);
  const unsigned long long group = ((1ull << LG) - 1) << base;
  const uint64_t none = j & 1 ? pack_ids(0, 0, tag) : pack_ids(-1, -1, tag);
  const uint64_t pad = pack_dev(__builtin_huge_valf(), -1, tag), no_arc = pack_arc(0.f, pass);
  uint64_t *rec = node + (size_t)c * NW;
  Polls<TICKETS, SWEEP_FORWARD> polls(wt);
  // own hop: lanes 0 and 1 of the group; arrivals through the arcs: lane j's
  // input.  Where some are missing, one lane first polls the own hop of the
  // turn's last cell, then all missing words are loaded together
  uint64_t ow = j < 2 ? pub_ld(rec + j) : none;
  const bool own_a = KM > 1 && j < n;
  uint64_t aw = own_a ? pub_ld(fa + t0 + j) : no_arc;
  if (__ballot(tag_lo(ow) != tag || arc_pass(aw) != pass)) {
    const uint64_t *last = node + (size_t)last_c * NW + 1;
    do {
      uint64_t lastw;
      do lastw = lane == 0 ? pub_ld(last) : none;
      while (polls.missing(tag_lo(lastw) != tag));
      do {
        if (tag_lo(ow) != tag) ow = pub_ld(rec + j);
        if (arc_pass(aw) != pass) aw = pub_ld(fa + t0 + j);
      } while (polls.missing(tag_lo(ow) != tag || arc_pass(aw) != pass));
    } while (polls.resume(tag_lo(ow) != tag || arc_pass(aw) != pass));
    if (polls.leave) return false;
  }
  const int pred = __shfl((int)(uint32_t)(ow >> 32), base, 64);
  const bool chain = pred >= tp.n_start;
  const uint64_t *p = node + (size_t)(chain ? pred - tp.n_start : 0) * NW;
  uint64_t hw = chain && j < HOP_WORDS - 2 ? pub_ld(p + j) : none;
  uint64_t lw = KM > 1 && chain && j < KM ? pub_ld(p + HOP_WORDS + j) : pad;
  uint32_t cd = j == 0 ? pub_ld(cdep + pred) : tag << 30;
  do {
    while (polls.missing(tag_lo(hw) != tag || tag_hi(lw) != tag || cd >> 30 != tag)) {
      if (tag_lo(hw) != tag) hw = pub_ld(p + j);
      if (tag_hi(lw) != tag) lw = pub_ld(p + HOP_WORDS + j);
      if (cd >> 30 != tag) cd = pub_ld(cdep + pred);
    }
  } while (polls.resume(tag_lo(hw) != tag || tag_hi(lw) != tag || cd >> 30 != tag));
  if (polls.leave) return false;
  if (on && j < HOP_WORDS - 2) pub_st(rec + 2 + j, hw);
  if (on && j == 0) pub_st(cdep + tp.n_start + c, ((cd + 1) & ID_MASK) | tag << 30);
  if constexpr (KM > 1) {
    Dev<float> e = unpack_dev(lw);
    const int arg = __shfl(id30((uint32_t)ow), base, 64) - t0;
    const int nmax = wave_max_int(n);
    const float a = arc_arrival(aw);
    float best = __shfl(a, base + (arg & (LG - 1)), 64);
    if (nmax > LG) {
      bool go = true;
      // (every lane of the wave waits for all of them)
      auto arc = [&](int i) {
        uint64_t w;
        do {
          do w = i < n ? pub_ld(fa + t0 + i) : no_arc;
          while (polls.missing(arc_pass(w) != pass));
        } while (polls.resume(arc_pass(w) != pass));
        go = !polls.leave;
        return arc_arrival(w);
      };
      const float far = arc(arg >= LG ? arg : n);
      if (arg >= LG) best = far;
      if (go) e = absorb_wide<float, KM>(e, best, n, nmax, arg, t0, group, go, arc);
      if (!go) return false;
    }
    int shift, rank;
    const float d = j < n && j != arg && best - a < __builtin_huge_valf() ? best - a : __builtin_huge_valf();
    list_ranks(e.cost, d, j, min(nmax, LG), group, [&](int i) { return __shfl(d, base + i, 64); }, shift, rank);
    if (on && d < __builtin_huge_valf() && rank < KM) pub_st(rec + HOP_WORDS + rank, pack_dev(d, t0 + j, tag));
    if (on && j < KM && j + shift < KM) pub_st(rec + HOP_WORDS + j + shift, pack_dev(e.cost, e.sink, tag));
  }
  return true;
}

// node records of the cells of turns w0, w0 + W, ..., or (TICKETS) of those that
// tickets give: turn q takes turn[q].y cells from turn[q].x on, at most
// 64 / list_lanes, of one level (two cells of one turn never wait for each
// other).  False if the wave left its share.
template <typename T, int KM, bool TICKETS>
__device__ __forceinline__ bool flow_lists(const Topo &tp, const int2 *__restrict__ turn, int turns, int w0, int W,
                                           uint32_t *__restrict__ cdep,
                                           uint64_t *__restrict__ node, const uint64_t *__restrict__ fa, uint32_t pass,
                                           const Waits<SWEEP_FORWARD> &wt) {
  static_assert(KM == 1 || sizeof(T) == 4, "double-precision lists are not published");
  const int g = wave_lane() / list_lanes(KM);
  // (spare groups repeat the turn's last cell and store nothing)
  auto cell = [&](int2 u) { return u.x + min(g, u.y - 1); };
  if constexpr (TICKETS) {
    for (int q; (q = take_ticket(&wt.share()->ticket[1])) < turns;) {
      const int2 u = turn[q];
      const int c = cell(u), t0 = tp.comb_inptr[c];
      list_turn_of<T, KM, true>(tp, c, g < u.y, u.x + u.y - 1, t0, tp.comb_inptr[c + 1] - t0, cdep, node, fa, pass, wt);
    }
    return true;
  }
  int q = w0;
  int2 u1 = make_int2(0, 1), u2 = u1;  // this wave's next two turns
  int nt0 = 0, nt1 = 0;                // the next turn's cells' input ranges
  if (q < turns) u1 = turn[q];
  if (q + W < turns) u2 = turn[q + W];
  if (q < turns) {
    nt0 = tp.comb_inptr[cell(u1)];
    nt1 = tp.comb_inptr[cell(u1) + 1];
  }
  for (; q < turns; q += W) {
    const int c = cell(u1);
    const bool on = g < u1.y;
    const int last_c = u1.x + u1.y - 1;
    const int t0 = nt0, n = nt1 - nt0;
    u1 = u2;
    if (q + W < turns) {
      nt0 = tp.comb_inptr[cell(u1)];
      nt1 = tp.comb_inptr[cell(u1) + 1];
    }
    if (q + 2 * W < turns) u2 = turn[q + 2 * W];
    if (!list_turn_of<T, KM, false>(tp, c, on, last_c, t0, n, cdep, node, fa, pass, wt)) return false;
  }
  return true;
}

// n_arr workgroups of arrival waves, the rest list waves; where shares are left,
// every workgroup takes tickets of both kinds, arrivals first (they wait for no
// list)
template <typename T, int KM>
__global__ void __launch_bounds__(256) k_forward_flow(Topo tp, LutView L, int n_arr, const int2 *__restrict__ turn,
                                                       int turns, const T *__restrict__ load,
                                                       const T *__restrict__ dnet, T *__restrict__ at,
                                                       T *__restrict__ slew, T *__restrict__ darc,
                                                       int32_t *__restrict__ crit, uint32_t *__restrict__ cdep,
                                                       uint64_t *__restrict__ node, uint64_t *__restrict__ fa,
                                                       uint64_t *__restrict__ fw, const uint32_t *__restrict__ d_tag,
                                                       Waits<SWEEP_FORWARD> wt) {
  extern __shared__ float4 s_lut4[];
  float *const s_lut = (float *)s_lut4;
  const int wpb = blockDim.x >> 6, wave = wave_id();
  begin_share(wt);
  const uint32_t pass = *d_tag;
  uint64_t *const arcs = KM > 1 ? fa : nullptr;
  bool done;
  if ((int)blockIdx.x < n_arr)
    done = flow_arrivals<T, false>(tp, L, s_lut, blockIdx.x * wpb + wave, n_arr * wpb, load, dnet, at, slew, darc, crit,
                                   node, node_words<T>(KM), arcs, fw, pass, wt);
  else
    done = flow_lists<T, KM, false>(tp, turn, turns, (blockIdx.x - n_arr) * wpb + wave,
                                    ((int)gridDim.x - n_arr) * wpb, cdep, node, fa, pass, wt);
  if (!__syncthreads_or(!done)) return;
  const SweepArgs &c = wt.args();
  const uint32_t again = *c.d_tag;
  flow_arrivals<T, true>(c.topo, c.lut, s_lut, 0, 0, (const T *)c.load, (const T *)c.dnet, (T *)c.at, (T *)c.slew,
                         (T *)c.darc, c.crit, c.node, node_words<T>(KM), KM > 1 ? c.flow_a : nullptr, c.flow_w, again, wt);
  flow_lists<T, KM, true>(c.topo, c.turn, c.turns, 0, 0, c.cdep, c.node, c.flow_a, again, wt);
}

// Backward: chunks from the last.  PULL: a sink lane loads the required time of
// its cell's output (the D pin of a flip-flop needs nothing), waiting only if
// it is not out yet, and stores its own; the driver lane publishes its own in
// fr.  PUSH: a sink lane loads its own required time, waiting likewise, and
// the driver lane publishes its cell's inputs', a consecutive run: one random
// read a sink where PULL has two and a random write, but three times the
// published words.  Many chunks per wave are bound by the random accesses and
// take PUSH, few by the chain and take PULL.  The required pass by itself, PUSH
// and PULL: 2M cells (120,623 chunks) 298 and 359 us, 1.4M (75,479) 215 and 232, 1M
// of 2 to 4 inputs (60,312) 190 and 200, 1M of 1 to 4 (53,901) 184 and 182, in
// double precision 193 and 197, 600,000 (32,352) 149 and 140, 200,000 (10,786) 119
// and 106.
constexpr int FANIN_AHEAD = 4;         // PUSH: inputs whose arcs are loaded before the wait
constexpr int PUSH_CHUNKS_PER_CU = 224;  // net chunks from which PUSH is taken (57,344 on 256 compute units)

static bool backward_pushes(const tdp_graph_s *g) {
  return g->topo.n_nm_chunks >= (long long)PUSH_CHUNKS_PER_CU * std::max(1, g->num_cu);
}

// One net chunk.  A wave that is to leave its share clears `done` and stores
// nothing (an early return instead costs 4 us at 200k cells).
template <typename T, bool PUSH, bool TICKETS>
__device__ __forceinline__ void backward_chunk(const Topo &tp, int4 rec, int k, const T *__restrict__ dnet_nm,
                                               const T *__restrict__ darc, T *rat, typename ReqWord<T>::type *words,
                                               const Waits<SWEEP_BACKWARD> &wt, bool &done) {
  using RW = typename ReqWord<T>::type;
  const int lane = wave_lane();
  const T inf = pos_inf<T>();
  const int p = rec.x;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  const bool sink = p >= 0 && lane != head, driver = p >= 0 && lane == head;
  const T dn = sink ? dnet_nm[k] : (T)0;
  T r = inf;
  if constexpr (PUSH) {
    const int nin = driver ? rec.w >> 16 : 0;
    const int t0 = rec.z;
    T da[FANIN_AHEAD];
#pragma unroll
    for (int j = 0; j < FANIN_AHEAD; ++j) da[j] = j < nin ? darc[t0 + j] : (T)0;
    // input sinks are numbered in level order and published from the top,
    // so the lowest one missing comes last
    const RW w = load_or_wait<true, TICKETS>(words, sink ? p : 0, sink, (RW)~(RW)0, wt, done);
    const T rt = ReqWord<T>::value(w);
    if (sink && rt != inf) r = rt - dn;
    r = seg_min(r, lane, head, tail);
    if (driver && done) {
      auto publish = [&](int j, T d) {
        const T ri = r != inf ? r - d : inf;
        pub_st(words + tp.M + t0 + j, pub_bits<T>(ri));
      };
#pragma unroll
      for (int j = 0; j < FANIN_AHEAD; ++j)
        if (j < nin) publish(j, da[j]);
      for (int j = FANIN_AHEAD; j < nin; ++j) publish(j, darc[t0 + j]);
    }
  } else {
    const int t = p - tp.M, vo = rec.z;
    const bool comb_in = sink && vo >= 0;
    const T da = comb_in ? darc[t] : (T)0;
    const T rq = sink && !comb_in ? rat[p] : (T)0;  // a D pin's, set at the endpoint
    // outputs are numbered in production order of the forward sweep, so the
    // backward sweep publishes the lowest one last
    const RW w = load_or_wait<true, TICKETS>(words, comb_in ? vo : 0, comb_in, (RW)~(RW)0, wt, done);
    if (sink && done) {
      const T rt = comb_in ? sink_required<T>(p, ReqWord<T>::value(w), da, rat) : rq;
      if (rt != inf) r = rt - dn;
    }
    r = seg_min(r, lane, head, tail);
    if (driver && done) pub_st(&words[p], pub_bits<T>(r));
  }
  if (driver && done) rat[p] = r;
}

template <typename T, bool PUSH>
__global__ void __launch_bounds__(256) k_backward_flow(Topo tp, const T *__restrict__ dnet_nm,
                                                        const T *__restrict__ darc, T *rat,
                                                        typename ReqWord<T>::type *fr, Waits<SWEEP_BACKWARD> wt) {
  using RW = typename ReqWord<T>::type;
  RW *const words = PUSH ? reinterpret_cast<RW *>(rat) : fr;
  const int lane = wave_lane();
  const int wpb = blockDim.x >> 6;
  const int W = gridDim.x * wpb;
  const int nch = tp.n_nm_chunks;
  int q = blockIdx.x * wpb + wave_id();
  int4 nrec = q < nch ? tp.nm_rec[(nch - 1 - q) * CHUNK + lane] : make_int4(-1, -1, -1, 0);
  begin_share(wt);
  bool done = true;
  for (; q < nch; q = done ? q + W : nch) {
    const int4 rec = nrec;
    if (q + W < nch) nrec = tp.nm_rec[(nch - 1 - q - W) * CHUNK + lane];
    backward_chunk<T, PUSH, false>(tp, rec, (nch - 1 - q) * CHUNK + lane, dnet_nm, darc, rat, words, wt, done);
  }
  if (!__syncthreads_or(!done)) return;
  const SweepArgs &c = wt.args();
  const int cn = c.topo.n_nm_chunks;
  while ((q = take_ticket(&wt.share()->ticket[0])) < cn) {
    const int k = (cn - 1 - q) * CHUNK + wave_lane();
    backward_chunk<T, PUSH, true>(c.topo, c.topo.nm_rec[k], k, (const T *)c.dnet_nm, (const T *)c.darc, (T *)c.rat,
                                  PUSH ? (RW *)c.rat : (RW *)c.flow_r, wt, done);
  }
}

// the backward sweep's words return to "not yet published": a new sweep
__global__ void k_backward_reset(uint32_t *words, size_t n, SweepShare *sh) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  fill_u32(words, n, ~0u, i, (size_t)gridDim.x * blockDim.x);
  if (i == 0) new_sweep(sh);
}

// --------------------------------------------------------------- export
template <typename T>
__global__ void __launch_bounds__(256) k_export(Topo tp, const T *__restrict__ at, const T *__restrict__ rat,
                                                 const T *__restrict__ slew,
                                                 const T *__restrict__ dnet, const T *__restrict__ load,
                                                 const T *__restrict__ darc, double *o_at, double *o_rat,
                                                 double *o_slack, double *o_slew, double *o_dnet,
                                                 double *o_load, double *o_darc, int net_model) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= tp.P) return;
  const int i = tp.ext_pin_int[p];
  const bool sink = i >= tp.M;
  const int t = i - tp.M;
  if (o_at) o_at[p] = (double)at[i];
  if (o_rat) o_rat[p] = (double)rat[i];
  if (o_slack) o_slack[p] = (double)(rat[i] != pos_inf<T>() ? rat[i] - at[i] : pos_inf<T>());
  if (o_slew) o_slew[p] = (double)(sink ? sink_slew<T>(net_model, slew[tp.snk_drv[t]], dnet[t]) : slew[i]);
  if (o_dnet) o_dnet[p] = sink ? (double)dnet[t] : 0.0;
  if (o_load) o_load[p] = sink ? 0.0 : (double)load[i];
  if (o_darc) o_darc[p] = (sink && t < tp.A) ? (double)darc[t] : 0.0;
}

__global__ void k_export_crit(Topo tp, const int32_t *__restrict__ crit, int32_t *__restrict__ out) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= tp.N) return;
  const int ci = tp.cell_int[cell];
  out[cell] = ci >= 0 ? crit[ci] : -1;
}

// --------------------------------------------------------------- launchers
static inline int nblk(long long n, int b) { return n > 0 ? (int)((n + b - 1) / b) : 1; }

static inline size_t lut_bytes(const LutView &L) { return sizeof(float4) * (size_t)L.n4; }

template <typename T, int KM>
static void launch_forward(tdp_graph g, int ch0, int ch1, int lc0, int lc1, const IncFlags &inc, hipStream_t s) {
  const Topo &tp = g->topo;
  const int n_arr = ch1 > ch0 ? nblk(ch1 - ch0, 4) : 0;
  const int n_lst = lc1 > lc0 ? nblk((long long)(lc1 - lc0) * list_lanes(KM), 256) : 0;
  if (n_arr + n_lst == 0) return;
  hipLaunchKernelGGL((k_forward<T, KM>), dim3(n_arr + n_lst), dim3(256), n_arr ? lut_bytes(g->lut) : 0, s, tp,
                     g->lut, ch0, ch1, n_arr, lc0, lc1, (const T *)g->load, (const T *)g->dnet, (T *)g->at,
                     (T *)g->slew, (V2<T> *)g->drv_as, (T *)g->darc, g->crit, g->cdep, g->node, (T *)g->fw_a,
                     g->d_tag, inc);
}

// arrivals of chunks [ch0, ch1) and the lists of cells [lc0, lc1), the level
// before
template <typename T>
static void forward_level(tdp_graph g, int ch0, int ch1, int lc0, int lc1, const IncFlags &inc, hipStream_t s) {
  switch (g->side_k) {
    case 1: launch_forward<T, 1>(g, ch0, ch1, lc0, lc1, inc, s); break;
    case 2: launch_forward<T, 2>(g, ch0, ch1, lc0, lc1, inc, s); break;
    case 4: launch_forward<T, 4>(g, ch0, ch1, lc0, lc1, inc, s); break;
    case 8: launch_forward<T, 8>(g, ch0, ch1, lc0, lc1, inc, s); break;
    case 16: launch_forward<T, 16>(g, ch0, ch1, lc0, lc1, inc, s); break;
    default: launch_forward<T, 32>(g, ch0, ch1, lc0, lc1, inc, s); break;
  }
}

// the per-level forward sweep over every level (incremental: with flags)
template <typename T>
static void forward_levels(tdp_graph g, const IncFlags &inc, hipStream_t s) {
  const Topo &tp = g->topo;
  int lc0 = 0, lc1 = 0;  // cells of the previous non-empty level, whose lists are due
  for (int l = 1; l <= tp.D; ++l) {
    const int ch0 = g->lv.fw_lvl[l - 1], ch1 = g->lv.fw_lvl[l];
    if (ch1 <= ch0) continue;
    forward_level<T>(g, ch0, ch1, lc0, lc1, inc, s);
    lc0 = g->lv.lvl[l - 1];
    lc1 = g->lv.lvl[l];
  }
  forward_level<T>(g, 0, 0, lc0, lc1, inc, s);
}

// Arrival workgroups: flow_per_cu per compute unit; list workgroups: three
// times that (a turn of a list wave waits longer and holds fewer cells than a
// chunk).  With 1 + 3 per compute unit the sweep takes 152 us at 200k cells
// (k = 10), 329 at 1M (k = 10), 465 at 2M (k = 8); with 1 + 2, 153, 385 and 571;
// with 1 + 4, 190, 385 and 480 (the waiting waves' polls get in the way); with
// 2 + 3, 154, 330 and 561.
constexpr int LIST_PER_ARR = 3;

template <typename T, int KM>
static void launch_forward_flow(tdp_graph g, hipStream_t s) {
  const Topo &tp = g->topo;
  const int w = g->flow_waves;
  const int occ = occupancy(reinterpret_cast<const void *>(&k_forward_flow<T, KM>), g->occ_fw, w, lut_bytes(g->lut));
  const int pa = std::max(1, std::min(occ / (1 + LIST_PER_ARR), g->flow_per_cu));
  const int na = resident_blocks(g, pa, w, tp.n_fw_chunks);
  const int nl = resident_blocks(g, std::min(occ - pa, LIST_PER_ARR * pa), w, g->n_turns);
  hipLaunchKernelGGL((k_forward_flow<T, KM>), dim3(na + nl), dim3(64 * w), lut_bytes(g->lut), s, tp, g->lut, na,
                     g->list_turn, g->n_turns,
                     (const T *)g->load, (const T *)g->dnet, (T *)g->at, (T *)g->slew, (T *)g->darc, g->crit, g->cdep,
                     g->node, g->flow_a, g->flow_w, g->d_tag, sweep_waits<SWEEP_FORWARD>(g));
}

template <typename T>
static void forward_flow(tdp_graph g, hipStream_t s) {
  if constexpr (sizeof(T) == 8) return launch_forward_flow<double, 1>(g, s);
  switch (g->side_k) {
    case 1: launch_forward_flow<float, 1>(g, s); break;
    case 2: launch_forward_flow<float, 2>(g, s); break;
    case 4: launch_forward_flow<float, 4>(g, s); break;
    case 8: launch_forward_flow<float, 8>(g, s); break;
    case 16: launch_forward_flow<float, 16>(g, s); break;
    default: launch_forward_flow<float, 32>(g, s); break;
  }
}

// net pass: pin positions, net delays, driver loads, start points (and the
// reset of the dataflow words in trailing workgroups).  sweep: an arrival sweep
// that writes every node record follows (a new tag)
template <typename T>
static void netpass_launch(tdp_graph g, const float *x, const float *y, const FlowInit &fl, bool sweep,
                           hipStream_t s) {
  // (a forward grid publishes through its own words and leaves drv_as and fw_a as they are)
  const Topo &tp = g->topo;
  const NetModel<T> nm = net_model<T>(g);
  const bool tree = g->lut.net_model == 2;
  const T *tree_wl = tree ? (const T *)g->tree.wl : nullptr;
  pack_xy(x, y, g->xy, tp.N, s, g->d_err + 1, ++g->pos_gen, g->d_err, g->d_tag,
          sweep ? g->d_tag + 2 : nullptr, fl.w ? 1u : 0u);
  const auto k_np = tree ? k_netpass<T, true> : k_netpass<T, false>;
  hipLaunchKernelGGL(k_np, dim3(nblk(tp.n_nm_chunks, 4) + fl.reset_blocks),
                     dim3(256), 0, s, tp, g->lut, g->xy, nm,
                     (T)g->c, (T)g->input_slew, (T)g->clock_slew, (T *)g->load, (T *)g->dnet, (T *)g->dnet_nm,
                     g->cxy_nm, (T *)g->at, (T *)g->slew, (V2<T> *)g->drv_as, g->cdep, fl);
  // nets wider than a chunk: their trees one thread per net first
  if (tp.n_big > 0 && tree) tree_net_impl<T>(g, g->tree, x, y, (T *)g->dnet, tp.big_net, tp.n_big, s);
  if (tp.n_big > 0)
    hipLaunchKernelGGL(k_netpass_big<T>, dim3(nblk(tp.n_big, 64)), dim3(64), 0, s, tp, g->lut, x, y, nm, tree_wl,
                       (T)g->c, (T)g->input_slew, (T)g->clock_slew, (T *)g->load, (T *)g->dnet, (T *)g->at,
                       (T *)g->slew, (V2<T> *)g->drv_as, g->cdep, fl);
}

template <typename T, bool SLACK>
static void endpoint_launch(tdp_graph g, hipStream_t s) {
  const Topo &tp = g->topo;
  hipLaunchKernelGGL((k_endpoint<T, SLACK>), dim3(g->n_ep_jobs), dim3(256), 0, s, tp, g->d_ep_base, g->ep_jobs,
                     g->d_inst_req, (const T *)g->dnet, (T *)g->at, (T *)g->rat, (T *)g->ep_slack,
                     g->red_ep, g->ep_counts, g->summary);
}

template <typename T>
void ep_reduce_impl(tdp_graph g, hipStream_t s) {
  endpoint_launch<T, false>(g, s);
}

template <typename T>
void netpass_impl(tdp_graph g, const float *x, const float *y, hipStream_t s) {
  FlowInit fl;
  fl.err = g->d_err;
  fl.tag = g->d_tag;
  netpass_launch<T>(g, x, y, fl, false, s);
}

// Which sweeps run as resident dataflow grids.  sweep_mode 1 and 2: both; 3:
// the backward one only; 4 (the choice for graphs that modes 1-3 do not take:
// double precision, or a net wider than a chunk): each that the graph allows.
// A published deviation is one word, so lists in double precision stay with
// the per-level launches; so do required times where a net is wider than a
// chunk.  The grids win at every size measured (forward / backward us: 2k
// cells, k = 10, 45 / 28 against 81 / 58; 200k 149 / 98 against 268 / 199; 2M,
// k = 8, 462 / 286 against 682 / 557): no kernel boundary per level, static data
// loaded ahead, and lists off the arrivals' way.
static bool flow_forward(const tdp_graph_s *g) {
  return g->sweep_mode == 1 || g->sweep_mode == 2 || (g->sweep_mode == 4 && g->fw_flow_ok);
}
static bool flow_backward(const tdp_graph_s *g) {
  return (g->sweep_mode >= 1 && g->sweep_mode <= 3) || (g->sweep_mode == 4 && g->bw_flow_ok);
}

// the words that the backward sweep publishes: input sinks' required times in
// place (PUSH), or drivers' in an array of their own
template <typename T>
static T *backward_words(tdp_graph g, int &n) {
  const bool push = backward_pushes(g);
  n = push ? g->topo.A : g->topo.M;
  return push ? (T *)g->rat + g->topo.M : (T *)g->flow_r;
}

// arrivals: net pass, forward sweep, endpoint slacks and WNS / TNS
template <typename T>
void sta_arrivals_impl(tdp_graph g, const float *x, const float *y, bool required, hipStream_t s) {
  const Topo &tp = g->topo;
  const NetModel<T> nm = net_model<T>(g);
  const bool flow = flow_forward(g), bflow = required && flow_backward(g);
  FlowInit fl;
  fl.err = g->d_err;
  fl.tag = g->d_tag;
  if (flow) {
    fl.w = g->flow_w;
    fl.node = g->node;
    fl.words = node_words<T>(g->side_k);
    fl.cd = g->cdep;
    fl.seed = g->sweep_mode == 2 ? 0 : 1;
    fl.fw = g->share + SWEEP_FORWARD;
  }
  if (bflow) {
    fl.r = backward_words<T>(g, fl.nr);
    fl.bw = g->share + SWEEP_BACKWARD;
  }
  fl.reset_blocks = flow ? 1024 : (bflow ? 64 : 0);
  prof_begin(g, TDP_STAGE_NETPASS, s);
  netpass_launch<T>(g, x, y, fl, true, s);
  g->flow_r_clear = bflow;
  prof_end(g, TDP_STAGE_NETPASS, s);
  prof_begin(g, TDP_STAGE_FORWARD, s);
  if (flow) {
    forward_flow<T>(g, s);
  } else {
    forward_levels<T>(g, IncFlags{}, s);
  }
  prof_end(g, TDP_STAGE_FORWARD, s);
  prof_begin(g, TDP_STAGE_ENDPOINT, s);
  endpoint_launch<T, true>(g, s);
  prof_end(g, TDP_STAGE_ENDPOINT, s);
}

// ---------------------------------------------------- incremental update
// forward chunk of every combinational input; net chunk of every driver
__global__ void k_inc_maps(Topo tp, int32_t *__restrict__ snk_chunk, int32_t *__restrict__ drv_nm_chunk) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long nf = (long long)tp.n_fw_chunks * CHUNK, nn = (long long)tp.n_nm_chunks * CHUNK;
  if (k < nf) {
    const int t = tp.fw_rec[k].x;
    if (t >= 0) snk_chunk[t] = (int)(k / CHUNK);
  } else if (k < nf + nn) {
    const long long q = k - nf;
    const int4 rec = tp.nm_rec[q];
    if (rec.x >= 0 && (int)(q % CHUNK) == (rec.w & 63)) drv_nm_chunk[rec.x] = (int)(q / CHUNK);
  }
}

// {arrival, transition} pairs of the combinational drivers from the two
// arrays, and each input's arrival through its arc (the same sum the
// arrival job forms), where the last forward sweep kept neither: the device
// knows (`stale`), since a captured pass may have run since the host last looked
template <typename T>
__global__ void k_pack_as(Topo tp, const uint32_t *__restrict__ stale, const T *__restrict__ at,
                          const T *__restrict__ slew, const T *__restrict__ darc, V2<T> *__restrict__ as,
                          T *__restrict__ fw_a) {
  if (!*stale) return;
  const int nth = gridDim.x * blockDim.x, i0 = blockIdx.x * blockDim.x + threadIdx.x;
  for (int i = i0; i < tp.n_comb; i += nth) as[tp.n_start + i] = v2<T>(at[tp.n_start + i], slew[tp.n_start + i]);
  for (int i = i0; i < tp.A; i += nth) fw_a[i] = at[tp.M + i] + darc[i];
}

// the error word of an incremental update: as it starts from the values of the
// last pass, a sweep that gave up there stays noted until a full update
__global__ void k_inc_begin(int32_t *err) { *err &= 2; }

// the net chunks that hold a moved cell's pins: its output's net and the nets
// of its inputs (bit 2 of err: an id outside [0, N))
__global__ void k_inc_mark(Topo tp, const int32_t *__restrict__ cells, int n, const int32_t *__restrict__ drv_nm_chunk,
                           int32_t *__restrict__ nm, int32_t epoch, int32_t *__restrict__ err) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int e = cells[i];
  if (e < 0 || e >= tp.N) {
    atomicOr(err, 4);
    return;
  }
  const int ci = tp.cell_int[e];
  auto mark = [&](int u) { nm[drv_nm_chunk[u]] = epoch; };
  if (ci >= 0) {
    mark(tp.n_start + ci);
    for (int t = tp.comb_inptr[ci]; t < tp.comb_inptr[ci + 1]; ++t) mark(tp.snk_drv[t]);
  } else {
    const int f = -ci - 1;
    mark(tp.n_pi + f);
    mark(tp.snk_drv[tp.A + f]);
  }
}

template <typename T>
void sta_arrivals_incremental_impl(tdp_graph g, const float *x, const float *y, const int32_t *cells, int n,
                                   hipStream_t s) {
  const Topo &tp = g->topo;
  const NetModel<T> nm = net_model<T>(g);
  IncFlags inc;
  inc.epoch = g->inc_epoch;
  inc.arr = g->inc_arr;
  inc.lst = g->inc_lst;
  inc.drv_chg = g->inc_drv_chg;
  inc.drv_lchg = g->inc_drv_lchg;
  inc.snk_chunk = g->inc_snk_chunk;
  inc.nm = g->inc_nm;
  prof_begin(g, TDP_STAGE_NETPASS, s);
  if (g->fw_flow_ok && tp.n_comb > 0)
    hipLaunchKernelGGL(k_pack_as<T>, dim3(std::min(2048, nblk(std::max(tp.n_comb, tp.A), 256))),
                       dim3(256), 0, s, tp, g->d_tag + 2, (const T *)g->at, (const T *)g->slew, (const T *)g->darc,
                       (V2<T> *)g->drv_as, (T *)g->fw_a);
  hipLaunchKernelGGL(k_inc_begin, dim3(1), dim3(1), 0, s, g->d_err);
  if (n > 0)
    hipLaunchKernelGGL(k_inc_mark, dim3(nblk(n, 256)), dim3(256), 0, s, tp, cells, n, g->inc_drv_nm_chunk,
                       g->inc_nm, inc.epoch, g->d_err);
  pack_xy(x, y, g->xy, tp.N, s, g->d_err + 1, ++g->pos_gen, nullptr, nullptr, g->d_tag + 2, 0u);
  // (every net fits a chunk here: graphs with wider nets take full updates)
  const auto k_npm = g->lut.net_model == 2 ? k_netpass_marked<T, true> : k_netpass_marked<T, false>;
  if (n > 0)
    hipLaunchKernelGGL(k_npm, dim3(nblk(tp.n_nm_chunks, 4)),
                       dim3(256), 0, s, tp, g->lut, g->xy, nm, (T)g->c,
                       (T)g->input_slew, (T)g->clock_slew, (T *)g->load, (T *)g->dnet, (T *)g->dnet_nm, g->cxy_nm,
                       (T *)g->at, (T *)g->slew, (V2<T> *)g->drv_as, g->cdep, inc);
  prof_end(g, TDP_STAGE_NETPASS, s);
  prof_begin(g, TDP_STAGE_FORWARD, s);
  forward_levels<T>(g, inc, s);
  prof_end(g, TDP_STAGE_FORWARD, s);
  prof_begin(g, TDP_STAGE_ENDPOINT, s);
  endpoint_launch<T, true>(g, s);
  prof_end(g, TDP_STAGE_ENDPOINT, s);
}

void inc_maps(tdp_graph g, hipStream_t s) {
  const Topo &tp = g->topo;
  const long long total = ((long long)tp.n_fw_chunks + tp.n_nm_chunks) * CHUNK;
  hipLaunchKernelGGL(k_inc_maps, dim3(nblk(total, 256)), dim3(256), 0, s, tp, g->inc_snk_chunk, g->inc_drv_nm_chunk);
}

template <typename T>
void sta_required_impl(tdp_graph g, hipStream_t s) {
  const Topo &tp = g->topo;
  const bool flow = flow_backward(g);
  prof_begin(g, TDP_STAGE_BACKWARD, s);
  if (flow) {
    // the words are reset by the arrival pass of the same call; a call of its
    // own resets them here
    int nr = 0;
    T *const words = backward_words<T>(g, nr);
    if (!g->flow_r_clear)
      hipLaunchKernelGGL(k_backward_reset, dim3(256), dim3(256), 0, s, reinterpret_cast<uint32_t *>(words),
                         (size_t)nr * (sizeof(T) / 4), g->share + SWEEP_BACKWARD);
    g->flow_r_clear = false;
    // twice flow_per_cu: 346 us against 379 at 2M cells, no difference at 200k
    const int w = g->flow_waves;
    const bool push = backward_pushes(g);
    const void *const kern = push ? reinterpret_cast<const void *>(&k_backward_flow<T, true>)
                                  : reinterpret_cast<const void *>(&k_backward_flow<T, false>);
    const int nb = resident_blocks(g, std::min(occupancy(kern, g->occ_bw, w, 0), 2 * g->flow_per_cu), w,
                                   tp.n_nm_chunks);
    using RW = typename ReqWord<T>::type;
    if (push)
      hipLaunchKernelGGL((k_backward_flow<T, true>), dim3(nb), dim3(64 * w), 0, s, tp, (const T *)g->dnet_nm,
                         (const T *)g->darc, (T *)g->rat, (RW *)nullptr, sweep_waits<SWEEP_BACKWARD>(g));
    else
      hipLaunchKernelGGL((k_backward_flow<T, false>), dim3(nb), dim3(64 * w), 0, s, tp, (const T *)g->dnet_nm,
                         (const T *)g->darc, (T *)g->rat, (RW *)g->flow_r, sweep_waits<SWEEP_BACKWARD>(g));
    prof_end(g, TDP_STAGE_BACKWARD, s);
    return;
  }
  for (int l = tp.D; l >= 0; --l) {
    const int ch0 = g->lv.nm_lvl[l], ch1 = g->lv.nm_lvl[l + 1];
    if (ch1 > ch0)
      hipLaunchKernelGGL(k_backward<T>, dim3(nblk(ch1 - ch0, 4)), dim3(256), 0, s, tp, ch0, ch1,
                         (const T *)g->dnet_nm, (const T *)g->darc, (T *)g->rat);
    const int b0 = g->lv.big_lvl[l], b1 = g->lv.big_lvl[l + 1];
    if (b1 > b0)
      hipLaunchKernelGGL(k_backward_big<T>, dim3(nblk(b1 - b0, 64)), dim3(64), 0, s, tp, b0, b1, (const T *)g->dnet,
                         (const T *)g->darc, (T *)g->rat);
  }
  prof_end(g, TDP_STAGE_BACKWARD, s);
}

template <typename T>
void sta_export_impl(tdp_graph g, double *at, double *rat, double *slack, double *slew, double *dnet,
                     double *load, double *darc, hipStream_t s) {
  const Topo &tp = g->topo;
  hipLaunchKernelGGL(k_export<T>, dim3(nblk(tp.P, 256)), dim3(256), 0, s, tp, (const T *)g->at,
                     (const T *)g->rat, (const T *)g->slew, (const T *)g->dnet,
                     (const T *)g->load, (const T *)g->darc, at, rat, slack, slew, dnet, load, darc,
                     g->lut.net_model);
}

void sta_export_crit(tdp_graph g, int32_t *out, hipStream_t s) {
  hipLaunchKernelGGL(k_export_crit, dim3(nblk(g->topo.N, 256)), dim3(256), 0, s, g->topo, g->crit, out);
}

template void ep_reduce_impl<float>(tdp_graph, hipStream_t);
template void ep_reduce_impl<double>(tdp_graph, hipStream_t);
template void netpass_impl<float>(tdp_graph, const float *, const float *, hipStream_t);
template void netpass_impl<double>(tdp_graph, const float *, const float *, hipStream_t);
template void sta_arrivals_incremental_impl<float>(tdp_graph, const float *, const float *, const int32_t *, int,
                                                   hipStream_t);
template void sta_arrivals_incremental_impl<double>(tdp_graph, const float *, const float *, const int32_t *, int,
                                                    hipStream_t);
template void sta_arrivals_impl<float>(tdp_graph, const float *, const float *, bool, hipStream_t);
template void sta_arrivals_impl<double>(tdp_graph, const float *, const float *, bool, hipStream_t);
template void sta_required_impl<float>(tdp_graph, hipStream_t);
template void sta_required_impl<double>(tdp_graph, hipStream_t);
template void sta_export_impl<float>(tdp_graph, double *, double *, double *, double *, double *, double *,
                                     double *, hipStream_t);
template void sta_export_impl<double>(tdp_graph, double *, double *, double *, double *, double *, double *,
                                      double *, hipStream_t);

}  // namespace tdp
