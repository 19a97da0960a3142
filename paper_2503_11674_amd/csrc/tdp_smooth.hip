// Differentiable objectives: a log-sum-exp smoothed TNS with its adjoint, and
// weighted-average wirelength.  Both give gradients on cell positions with a
// fixed summation order per cell (terms per pin computed per net, then
// gathered over the cell's own pins; no floating-point atomics).
//
// Smoothed TNS (not in the paper; this is its definition here): cell-arc
// delays and start-point arrivals are frozen from the last timing update, net
// delays follow the positions (the library's net model as a function of L,
// the Manhattan length).
//   sink t:          A(t) = A(drv) + dnet(t)
//   comb output o:   A(o) = m + g ln sum_j exp((a_j - m)/g), a_j = A(in_j) + d_arc(in_j)
//   endpoint e:      s(e) = (period - setup) - A(e)
//   value:           -g * sum_e softplus(-s(e)/g)
// The adjoint runs the levels top-down: dv/dA(e) = -sigmoid(-s(e)/g); an
// output passes its adjoint to input j in proportion to softmax_j(a/g); a
// driver collects the adjoints of its sinks (over the net chunks, as the
// required-time pass runs).  dv/d dnet(t) is the adjoint at
// t, and on a star net d dnet/dX_s = dnet'(L) sign(X_s - X_t) = -d dnet/dX_t
// (the spanning-tree model differentiates through its tree).  The net delays
// and the per-pin terms come from the net kernels of tdp_tree.hip.
//
// Weighted-average wirelength (the smoothed WL of Eq. 1): per net and axis,
// sum x e^{x/g} / sum e^{x/g} - sum x e^{-x/g} / sum e^{-x/g}, with the
// exponents shifted by the net's max and min.
#include "tdp_flow.h"
#include "tdp_impl.h"
#include "tdp_look.h"
#include "tdp_prims.h"
#include "tdp_wave.h"

namespace tdp {

static inline int nb(long long n, int b) { return n > 0 ? (int)((n + b - 1) / b) : 1; }

// the smoothed sweeps' own error words, ST_ERR behind d_err's: this forward pass's and
// its backward passes', and one that stays set until a call has reported it (the
// next update clears the timing sweeps' word, and no smoothed call waits for its
// results)
__device__ __forceinline__ bool st_failed(const int32_t *err) {
  return pub_ld(reinterpret_cast<const uint32_t *>(err)) != 0;
}
__device__ __forceinline__ void st_report(int32_t *err) {
  if (st_failed(err)) pub_st(reinterpret_cast<uint32_t *>(err + 1), 1u);
}

template <typename T>
__device__ __forceinline__ T sgn(T v) {
  return (T)((v > (T)0) - (v < (T)0));
}

// start points' arrivals; every other driver's word, and every driver's
// adjoint, not yet
template <typename T>
__global__ void __launch_bounds__(256) k_st_start(Topo tp, const T *__restrict__ at, T *__restrict__ sa,
                                                   T *__restrict__ adj, int32_t *__restrict__ err,
                                                   SweepShare *__restrict__ share) {
  using RW = typename ReqWord<T>::type;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    err[0] = 0;
    new_sweep(share + SWEEP_ST_FORWARD);
    new_sweep(share + SWEEP_ST_BACKWARD);
  }
  for (int v = blockIdx.x * blockDim.x + threadIdx.x; v < tp.M; v += gridDim.x * blockDim.x) {
    reinterpret_cast<RW *>(sa)[v] = v < tp.n_start ? pub_bits<T>(at[v]) : ~(RW)0;
    reinterpret_cast<RW *>(adj)[v] = ~(RW)0;
  }
}

// A chunk's combinational cells, a lane per input (each cell a segment): the
// input's arrival through its arc (ai: its driver's arrival), the cell's
// log-sum-exp over its inputs by segment reductions, and each input's share of
// the output's adjoint, its softmax weight, for the backward sweep
template <typename T>
struct StCell {
  T a, out;
  __device__ __forceinline__ StCell(T ai, T dn, T da, bool valid, int lane, int head, int tail, T gam) {
    a = valid ? (ai + dn) + da : -pos_inf<T>();
    const T m = seg_max(a, lane, head, tail);
    const T sum = seg_sum(valid ? exp((a - m) / gam) : (T)0, lane, head, tail);
    out = m + gam * log(sum);
  }
  __device__ __forceinline__ T share(T gam) const { return exp((a - out) / gam); }
};

// one level's cells on the forward chunks
template <typename T>
__global__ void __launch_bounds__(256) k_st_fwd(Topo tp, int ch0, int ch1, T gam, const T *__restrict__ dnl,
                                                 const T *__restrict__ darc, T *__restrict__ sa) {
  const int lane = wave_lane();
  const int chunk = ch0 + blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= ch1) return;
  const int4 rec = tp.fw_rec[chunk * CHUNK + lane];
  const int t = rec.x;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  const bool valid = t >= 0;
  const StCell<T> c(valid ? sa[rec.y] : (T)0, valid ? dnl[t] : (T)0, valid ? darc[t] : (T)0, valid, lane, head, tail,
                    gam);
  if (valid && lane == head) sa[tp.n_start + rec.z] = c.out;
  if (valid) sa[tp.M + t] = c.share(gam);
}

// The whole forward sweep on a resident grid (see the dataflow sweeps of the
// timing pass): wave w takes chunks w, w + W, ... in level order, waits for its
// drivers' words and publishes its cells'.  Bound by the chain of levels: 157 us
// at 1M cells, 80 levels, against 312 with a launch per level.
template <typename T, bool TICKETS>
__device__ __forceinline__ void st_fwd_chunk(const Topo &tp, int4 rec, T gam, const T *__restrict__ dnl,
                                             const T *__restrict__ darc, T *sa, const Waits<SWEEP_ST_FORWARD> &wt,
                                             bool &done) {
  using RW = typename ReqWord<T>::type;
  RW *words = reinterpret_cast<RW *>(sa);
  const int lane = wave_lane();
  const int t = rec.x;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  const bool valid = t >= 0;
  const T dn = valid ? dnl[t] : (T)0, da = valid ? darc[t] : (T)0;
  RW w;
  done = load_or_leave<false, TICKETS>(words, valid ? rec.y : 0, valid, (RW)~(RW)0, wt, w);
  if (!done) return;
  const StCell<T> c(ReqWord<T>::value(w), dn, da, valid, lane, head, tail, gam);
  if (valid && lane == head) pub_st(words + tp.n_start + rec.z, pub_bits<T>(c.out));
  if (valid) sa[tp.M + t] = c.share(gam);
}

template <typename T>
__global__ void __launch_bounds__(256) k_st_fwd_flow(Topo tp, T gam, const T *__restrict__ dnl,
                                                      const T *__restrict__ darc, T *sa, Waits<SWEEP_ST_FORWARD> wt) {
  const int lane = wave_lane(), wpb = blockDim.x >> 6;
  const int W = gridDim.x * wpb, nch = tp.n_fw_chunks;
  int q = blockIdx.x * wpb + wave_id();
  int4 nrec = q < nch ? tp.fw_rec[q * CHUNK + lane] : make_int4(-1, 0, 0, 0);
  begin_share(wt);
  bool done = true;
  for (; done && q < nch; q += W) {
    const int4 rec = nrec;
    if (q + W < nch) nrec = tp.fw_rec[(q + W) * CHUNK + lane];
    st_fwd_chunk<T, false>(tp, rec, gam, dnl, darc, sa, wt, done);
  }
  if (__syncthreads_or(!done)) {
    const SweepArgs &c = wt.args();
    while ((q = take_ticket(&wt.share()->ticket[0])) < c.topo.n_fw_chunks)
      st_fwd_chunk<T, true>(c.topo, c.topo.fw_rec[q * CHUNK + wave_lane()], gam, (const T *)c.st_dnet, (const T *)c.darc,
                            (T *)c.st_at, wt, done);
  }
  if (lane == 0) st_report(wt.err());
}

// endpoint values and adjoint seeds; the value summed by the last workgroup (not
// a number after a sweep that gave up)
template <typename T>
__global__ void __launch_bounds__(256) k_st_end(Topo tp, const double *__restrict__ inst_req, T gam,
                                                 const T *__restrict__ dnl, const T *__restrict__ sa,
                                                 T *__restrict__ adj, double *__restrict__ part,
                                                 uint32_t *__restrict__ ctr, double *__restrict__ val,
                                                 const int32_t *__restrict__ err) {
  __shared__ double sh[256];
  double acc = *err ? __builtin_nan("") : 0.0;
  for (int f = blockIdx.x * blockDim.x + threadIdx.x; f < tp.E; f += gridDim.x * blockDim.x) {
    const int t = tp.A + f;
    const T a = sa[tp.snk_drv[t]] + dnl[t];
    const T z = (a - (T)inst_req[tp.ff_inst[f]]) / gam;  // -slack / g
    const T sp = (z > 0 ? z : (T)0) + log1p(exp(-fabs(z)));
    acc += (double)(-gam * sp);
    adj[tp.M + t] = -(T)1 / ((T)1 + exp(-z));
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) pub_st(part + blockIdx.x, sh[0]);
  last_sum(ctr, gridDim.x, part, val);
}

// The adjoint of one level's nets (drivers at that level, top-down), a lane
// per net pin: a combinational-input sink takes its cell output's adjoint
// times its share (the output's level is higher, so it is final), an
// endpoint keeps the seed the endpoint kernel wrote; the driver collects its
// sinks' (a segment sum).
template <typename T>
__global__ void __launch_bounds__(256) k_st_bwd(Topo tp, int ch0, int ch1, const T *__restrict__ sa,
                                                 T *__restrict__ adj, T *__restrict__ adj_nm) {
  const int lane = wave_lane();
  const int chunk = ch0 + blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= ch1) return;
  const int4 rec = tp.nm_rec[chunk * CHUNK + lane];
  const int p = rec.x, vo = rec.z;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  T a = 0;
  if (p >= 0 && lane != head) {
    a = vo >= 0 ? adj[vo] * sa[p] : adj[p];
    adj_nm[chunk * CHUNK + lane] = a;
  }
  a = seg_sum(a, lane, head, tail);
  if (p >= 0 && lane == head) adj[p] = a;
}

// The whole backward sweep on a resident grid, in reverse level order (no net
// wider than a chunk): 147 us at 1M cells against 385 with a launch per level,
// which also gathered the arc, both arrivals and the exponential of each share.
// STAR: the pins' gradients under the star models as well, after the driver's
// adjoint is out: the waves wait for most of a level's time, and part of the
// gathers and the scatter fits in it (191 us at 1M cells against 147 + 82 in
// two launches; 46 against 44 + 6 at 50,000).  Otherwise the sinks' adjoints go
// to adj_nm for the spanning trees' launch.
template <typename T, bool STAR, bool TICKETS>
__device__ __forceinline__ void st_bwd_chunk(const Topo &tp, int4 rec, int k, const T *__restrict__ sa, T *adj,
                                             T *__restrict__ adj_nm, const float2 *__restrict__ xy,
                                             const NetModel<T> &nm, V2<T> *__restrict__ gp, const Waits<SWEEP_ST_BACKWARD> &wt,
                                             bool &done) {
  using RW = typename ReqWord<T>::type;
  RW *words = reinterpret_cast<RW *>(adj);
  const int lane = wave_lane();
  const int p = rec.x, vo = rec.z;
  const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
  const bool sink = p >= 0 && lane != head, comb_in = sink && vo >= 0;
  // a combinational input's share, an endpoint's seed
  const T share = sink ? (comb_in ? sa : adj)[p] : (T)0;
  float2 pos = make_float2(0.f, 0.f), off = pos;
  if constexpr (STAR) {
    if (rec.y >= 0) pos = xy[rec.y];
    off = make_float2(tp.nm_ox[k], tp.nm_oy[k]);
  }
  RW w;
  done = load_or_leave<true, TICKETS>(words, comb_in ? vo : 0, comb_in, (RW)~(RW)0, wt, w);
  if (!done) return;
  const T mine = comb_in ? ReqWord<T>::value(w) * share : share;
  const T a = seg_sum(mine, lane, head, tail);
  if (p >= 0 && lane == head) pub_st(words + p, pub_bits<T>(a));
  if constexpr (STAR) {
    // (driver - sink) per axis, a port's position as the base (see the net pass)
    const bool port = rec.y < 0;
    const T cx = port ? (T)off.x : (T)pos.x, cy = port ? (T)off.y : (T)pos.y;
    const T ox = port ? (T)0 : (T)off.x, oy = port ? (T)0 : (T)off.y;
    const T cxd = __shfl(cx, head, 64), cyd = __shfl(cy, head, 64);
    const T oxd = __shfl(ox, head, 64), oyd = __shfl(oy, head, 64);
    const T dx = (cxd - cx) + (oxd - ox), dy = (cyd - cy) + (oyd - oy);
    const T len = sink ? fabs(dx) + fabs(dy) : (T)0;
    const T gl = sink ? mine * nm.slope(len, nm.elmore ? (T)tp.type_cap[(rec.w >> 16) & 255] : (T)0) : (T)0;
    const T ex = gl * sgn(dx), ey = gl * sgn(dy);
    const T sx = seg_sum(ex, lane, head, tail), sy = seg_sum(ey, lane, head, tail);
    if (p >= 0) gp[p] = sink ? v2<T>(-ex, -ey) : v2<T>(sx, sy);
  } else {
    if (sink) adj_nm[k] = mine;
  }
}

template <typename T, bool STAR>
__global__ void __launch_bounds__(256) k_st_bwd_flow(Topo tp, const T *__restrict__ sa, T *adj,
                                                      T *__restrict__ adj_nm, const float2 *__restrict__ xy,
                                                      NetModel<T> nm, V2<T> *__restrict__ gp, Waits<SWEEP_ST_BACKWARD> wt) {
  const int lane = wave_lane(), wpb = blockDim.x >> 6;
  const int W = gridDim.x * wpb, nch = tp.n_nm_chunks;
  int q = blockIdx.x * wpb + wave_id();
  int4 nrec = q < nch ? tp.nm_rec[(nch - 1 - q) * CHUNK + lane] : make_int4(-1, -1, -1, 0);
  begin_share(wt);
  bool done = true;
  for (; done && q < nch; q += W) {
    const int4 rec = nrec;
    if (q + W < nch) nrec = tp.nm_rec[(nch - 1 - q - W) * CHUNK + lane];
    st_bwd_chunk<T, STAR, false>(tp, rec, (nch - 1 - q) * CHUNK + lane, sa, adj, adj_nm, xy, nm, gp, wt, done);
  }
  if (__syncthreads_or(!done)) {
    const SweepArgs &c = wt.args();
    const int cn = c.topo.n_nm_chunks;
    while ((q = take_ticket(&wt.share()->ticket[0])) < cn) {
      const int k = (cn - 1 - q) * CHUNK + wave_lane();
      st_bwd_chunk<T, STAR, true>(c.topo, c.topo.nm_rec[k], k, (const T *)c.st_at, (T *)c.st_adj, (T *)c.st_adj_nm,
                                  c.xy_st, nm, (V2<T> *)c.st_gp, wt, done);
    }
  }
  if (lane == 0) st_report(wt.err());
}

// the same for nets wider than a chunk, one thread per net
template <typename T>
__global__ void k_st_bwd_big(Topo tp, int i0, int i1, const T *__restrict__ sa, T *__restrict__ adj) {
  const int i = i0 + blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= i1) return;
  const int v = tp.big_net[i];
  T ab = 0;
  for (int k = tp.net_ptr[v]; k < tp.net_ptr[v + 1]; ++k) {
    const int t = tp.net_sink[k];
    const int p = tp.M + t;
    T a;
    if (t < tp.A) {
      a = adj[tp.n_start + tp.snk_comb[t]] * sa[p];
      adj[p] = a;
    } else {
      a = adj[p];
    }
    ab += a;
  }
  adj[v] = ab;
}

// gradient per cell: the sum of its pins' gradients (its output pin, then its
// input pins), which the net kernels computed per pin (not numbers after a
// sweep that gave up)
template <typename T>
__global__ void __launch_bounds__(256) k_st_grad(Topo tp, const V2<T> *__restrict__ gp, const double *__restrict__ gout,
                                                  float *__restrict__ gx, float *__restrict__ gy,
                                                  const int32_t *__restrict__ err) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= tp.N || tp.cell_fixed[cell]) return;
  const int ci = tp.cell_int[cell];
  int v, t0, t1;
  if (ci >= 0) {
    v = tp.n_start + ci;
    t0 = tp.comb_inptr[ci];
    t1 = tp.comb_inptr[ci + 1];
  } else {
    const int f = -ci - 1;
    v = tp.n_pi + f;
    t0 = tp.A + f;
    t1 = t0 + 1;
  }
  const V2<T> out = gp[v];
  T ax = out.x, ay = out.y;
  for (int t = t0; t < t1; ++t) {
    const V2<T> in = gp[tp.M + t];
    ax += in.x;
    ay += in.y;
  }
  const T go = *err ? (T)__builtin_nan("") : (T)*gout;
  gx[cell] += (float)(go * ax);
  gy[cell] += (float)(go * ay);
}

__global__ void __launch_bounds__(256) k_sum_parts2(int n, const double *__restrict__ part, double *__restrict__ out) {
  __shared__ double sh[256];
  double a = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) a += part[i];
  sh[threadIdx.x] = a;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *out = sh[0];
}

constexpr int RED_BLOCKS = 512;

// workgroups of a smoothed sweep's resident grid (dir 0 forward, 1 backward)
static int st_blocks(tdp_graph g, const void *kern, int dir, int chunks) {
  const int w = g->flow_waves, occ = occupancy(kern, g->occ_st[dir], w, 0);
  return resident_blocks(g, std::min(occ, 2 * g->flow_per_cu), w, chunks);
}

// Both sweeps run as resident grids unless sweep_mode 0 asks for a launch per
// level; backward, nets wider than a chunk do too.
template <typename T>
void stns_fwd_impl(tdp_graph g, const float *x, const float *y, float gamma, double *val, hipStream_t s) {
  const Topo &tp = g->topo;
  prof_begin(g, TDP_STAGE_STNS, s);
  const T gam = (T)gamma;
  st_net_fwd_impl<T>(g, x, y, (T *)g->st_dnet, s);
  hipLaunchKernelGGL(k_st_start<T>, dim3(std::min(2048, nb(tp.M, 256))), dim3(256), 0, s, tp, (const T *)g->at,
                     (T *)g->st_at, (T *)g->st_adj, g->d_err + ST_ERR, g->share);
  if (g->sweep_mode != 0) {
    const int w = g->flow_waves;
    hipLaunchKernelGGL(k_st_fwd_flow<T>,
                       dim3(st_blocks(g, reinterpret_cast<const void *>(&k_st_fwd_flow<T>), 0, tp.n_fw_chunks)),
                       dim3(64 * w), 0, s, tp, gam, (const T *)g->st_dnet, (const T *)g->darc, (T *)g->st_at,
                       sweep_waits<SWEEP_ST_FORWARD>(g));
  } else {
    for (int l = 1; l <= tp.D; ++l) {
      const int ch0 = g->lv.fw_lvl[l - 1], ch1 = g->lv.fw_lvl[l];
      if (ch1 > ch0)
        hipLaunchKernelGGL(k_st_fwd<T>, dim3(nb(ch1 - ch0, 4)), dim3(256), 0, s, tp, ch0, ch1, gam,
                           (const T *)g->st_dnet, (const T *)g->darc, (T *)g->st_at);
    }
  }
  hipLaunchKernelGGL(k_st_end<T>, dim3(std::min(128, nb(tp.E, 256))), dim3(256), 0, s, tp, g->d_inst_req, gam,
                     (const T *)g->st_dnet, (const T *)g->st_at, (T *)g->st_adj, g->red_loss, g->look_ctr + 8, val,
                     g->d_err + ST_ERR);
  g->st_gamma = gamma;
  g->st_x = x;
  g->st_y = y;
  g->stns_ready = true;
  prof_end(g, TDP_STAGE_STNS, s);
}

template <typename T>
void stns_bwd_impl(tdp_graph g, const double *gout, float *gx, float *gy, hipStream_t s) {
  const Topo &tp = g->topo;
  prof_begin(g, TDP_STAGE_STNS, s);
  const bool flow = g->sweep_mode != 0 && g->bw_flow_ok, star = g->lut.net_model != 2;
  if (flow) {
    const void *const kern = star ? reinterpret_cast<const void *>(&k_st_bwd_flow<T, true>)
                                  : reinterpret_cast<const void *>(&k_st_bwd_flow<T, false>);
    const dim3 grid(st_blocks(g, kern, 1, tp.n_nm_chunks)), block(64 * g->flow_waves);
    if (star)
      hipLaunchKernelGGL((k_st_bwd_flow<T, true>), grid, block, 0, s, tp, (const T *)g->st_at, (T *)g->st_adj,
                         (T *)nullptr, g->xy_st, net_model<T>(g), (V2<T> *)g->st_gp,
                         sweep_waits<SWEEP_ST_BACKWARD>(g));
    else
      hipLaunchKernelGGL((k_st_bwd_flow<T, false>), grid, block, 0, s, tp, (const T *)g->st_at, (T *)g->st_adj,
                         (T *)g->st_adj_nm, g->xy_st, net_model<T>(g), (V2<T> *)nullptr,
                         sweep_waits<SWEEP_ST_BACKWARD>(g));
  } else {
    for (int l = tp.D; l >= 0; --l) {
      const int ch0 = g->lv.nm_lvl[l], ch1 = g->lv.nm_lvl[l + 1];
      if (ch1 > ch0)
        hipLaunchKernelGGL(k_st_bwd<T>, dim3(nb(ch1 - ch0, 4)), dim3(256), 0, s, tp, ch0, ch1, (const T *)g->st_at,
                           (T *)g->st_adj, (T *)g->st_adj_nm);
      const int b0 = g->lv.big_lvl[l], b1 = g->lv.big_lvl[l + 1];
      if (b1 > b0)
        hipLaunchKernelGGL(k_st_bwd_big<T>, dim3(nb(b1 - b0, 64)), dim3(64), 0, s, tp, b0, b1, (const T *)g->st_at,
                           (T *)g->st_adj);
    }
  }
  // (no net wider than a chunk where the sweep was a grid)
  if (!(flow && star))
    st_net_grad_impl<T>(g, g->st_x, g->st_y, (const T *)g->st_adj, (const T *)g->st_adj_nm, s);
  hipLaunchKernelGGL(k_st_grad<T>, dim3(nb(tp.N, 256)), dim3(256), 0, s, tp, (const V2<T> *)g->st_gp, gout,
                     gx, gy, g->d_err + ST_ERR);
  prof_end(g, TDP_STAGE_STNS, s);
}

// ------------------------------------------------------------------- WA
// Coordinates enter relative to the net's max (the e^{x/g} side) and min (the
// e^{-x/g} side): d = x - max <= 0, e = x - min >= 0, so the weighted means
// and the (x - mean) terms stay small numbers in single precision.
//   WA = (max - min) + sum d a / sum a - sum e b / sum b,  a = e^{d/g}, b = e^{-e/g}
//   dWA/dx = a/sum a (1 + (d - sum d a / sum a)/g) - b/sum b (1 - (e - sum e b / sum b)/g)

// one axis for one lane of a chunked net; returns the net's WA on that axis.
// A pin's coordinate is (cell position c) + (offset o); differences are taken
// as (c_i - c_m) + (o_i - o_m), which keeps them exact to within the rounding
// of the result instead of carrying the rounding of c + o at die scale.
__device__ __forceinline__ float wa_lane(float c, float o, bool valid, int lane, int head, int tail, float ig,
                                         float &grad) {
  const float X = c + o;
  const float mx = seg_max_dpp(valid ? X : -3.0e38f, lane, head, tail);
  const float mn = seg_min_dpp(valid ? X : 3.0e38f, lane, head, tail);
  const int am = seg_min_dpp((valid && X == mx) ? lane : 64, lane, head, tail) & 63;
  const int an = seg_min_dpp((valid && X == mn) ? lane : 64, lane, head, tail) & 63;
  const float cm = __shfl(c, am, 64), om = __shfl(o, am, 64);
  const float cn = __shfl(c, an, 64), on = __shfl(o, an, 64);
  const float d = valid ? (c - cm) + (o - om) : 0.f, e = valid ? (c - cn) + (o - on) : 0.f;
  // exponents are <= 0 (d <= 0 <= e); the hardware exponential (2^(x log2 e))
  // has a relative error of about |x| 2^-24 plus a few units in the last
  // place, and terms with large |x| are negligible in the sums
  const float a = valid ? __expf(d * ig) : 0.f, b = valid ? __expf(-e * ig) : 0.f;
  const float sa = seg_sum_dpp(a, lane, head, tail), sda = seg_sum_dpp(a * d, lane, head, tail);
  const float sb = seg_sum_dpp(b, lane, head, tail), seb = seg_sum_dpp(b * e, lane, head, tail);
  const float ra = valid ? 1.f / sa : 0.f, rb = valid ? 1.f / sb : 0.f;  // sa, sb >= 1 (the extreme pin's term)
  const float fp = sda * ra, fm = seb * rb;
  grad = valid ? a * ra * (1.f + (d - fp) * ig) - b * rb * (1.f - (e - fm) * ig) : 0.f;
  return valid ? ((cm - cn) + (om - on)) + fp - fm : 0.f;
}

// chunked nets: value partials and the gradient of each pin (internal pin order)
// cxy (optional): the cell coordinates of every slot, gathered by the last
// timing update; otherwise they are gathered here from xy
__global__ void __launch_bounds__(256) k_wa_net(Topo tp, const float2 *__restrict__ xy,
                                                 const float2 *__restrict__ cxy, float gam,
                                                 float *__restrict__ gpin, double *__restrict__ part) {
  __shared__ double sh[256];
  double acc = 0.0;
  const float ig = 1.0f / gam;
  const int lane = wave_lane();
  const int stride = gridDim.x * 4;
  // each chunk's inputs are loaded one chunk ahead, before the current
  // chunk's stores: a wave's loads retire after its earlier stores, so a
  // load issued after them would wait for them
  auto fetch = [&](int chunk, int4 &rec, float2 &q, float &ox, float &oy) {
    const int k = chunk * CHUNK + lane;
    rec = tp.nm_rec[k];
    q = cxy ? cxy[k] : (rec.y >= 0 ? xy[rec.y] : make_float2(0.f, 0.f));
    ox = tp.nm_ox[k];
    oy = tp.nm_oy[k];
  };
  int chunk = blockIdx.x * 4 + (threadIdx.x >> 6);
  int4 nrec = make_int4(-1, -1, -1, 0);
  float2 nq = make_float2(0.f, 0.f);
  float nox = 0.f, noy = 0.f;
  if (chunk < tp.n_nm_chunks) fetch(chunk, nrec, nq, nox, noy);
  for (; chunk < tp.n_nm_chunks; chunk += stride) {
    const int4 rec = nrec;
    const float2 q = nq;
    const float ox = nox, oy = noy;
    if (chunk + stride < tp.n_nm_chunks) fetch(chunk + stride, nrec, nq, nox, noy);
    const int p = rec.x;
    const int head = rec.w & 63, tail = (rec.w >> 8) & 63;
    const bool valid = p >= 0;
    float gxp, gyp;
    const float wx = wa_lane(q.x, ox, valid, lane, head, tail, ig, gxp);
    const float wy = wa_lane(q.y, oy, valid, lane, head, tail, ig, gyp);
    if (valid) {
      gpin[2 * p] = gxp;
      gpin[2 * p + 1] = gyp;
      if (lane == head) acc += (double)wx + (double)wy;
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// nets wider than a chunk: one thread per net, same arithmetic
__global__ void __launch_bounds__(64) k_wa_big(Topo tp, const float2 *__restrict__ xy, float gam,
                                                float *__restrict__ gpin, double *__restrict__ part) {
  __shared__ double sh[64];
  double acc = 0.0;
  const float ig = 1.0f / gam;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < tp.n_big; i += gridDim.x * blockDim.x) {
    const int v = tp.big_net[i];
    const int b = tp.net_ptr[v], e = tp.net_ptr[v + 1];
    const int dc = tp.drv_cell[v];
    for (int axis = 0; axis < 2; ++axis) {
      const float *so = axis ? tp.snk_oy : tp.snk_ox;
      auto pc = [&](int cell) { return axis ? xy[cell].y : xy[cell].x; };
      const float pd = (dc >= 0 ? pc(dc) : 0.f) + (axis ? tp.drv_oy[v] : tp.drv_ox[v]);
      float mx = pd, mn = pd;
      for (int k = b; k < e; ++k) {
        const int t = tp.net_sink[k];
        const float q = pc(tp.snk_cell[t]) + so[t];
        mx = fmaxf(mx, q);
        mn = fminf(mn, q);
      }
      float sa = 0.f, sda = 0.f, sb = 0.f, seb = 0.f;
      for (int k = b - 1; k < e; ++k) {
        const float q = k < b ? pd : pc(tp.snk_cell[tp.net_sink[k]]) + so[tp.net_sink[k]];
        const float d = q - mx, ee = q - mn;
        const float a = expf(d * ig), bb = expf(-ee * ig);
        sa += a; sda += a * d; sb += bb; seb += bb * ee;
      }
      const float fp = sda / sa, fm = seb / sb;
      acc += (double)((mx - mn) + fp - fm);
      for (int k = b - 1; k < e; ++k) {
        const int t = k < b ? -1 : tp.net_sink[k];
        const float q = k < b ? pd : pc(tp.snk_cell[t]) + so[t];
        const float d = q - mx, ee = q - mn;
        const float a = expf(d * ig), bb = expf(-ee * ig);
        const float gr = a / sa * (1.f + (d - fp) * ig) - bb / sb * (1.f - (ee - fm) * ig);
        gpin[2 * (k < b ? v : tp.M + t) + axis] = gr;
      }
    }
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int o = 32; o > 0; o >>= 1) {
    if (threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

__global__ void __launch_bounds__(256) k_wa_cell(Topo tp, const float *__restrict__ gpin, float *__restrict__ gx,
                                                  float *__restrict__ gy) {
  const int cell = blockIdx.x * blockDim.x + threadIdx.x;
  if (cell >= tp.N || tp.cell_fixed[cell]) return;
  const int ci = tp.cell_int[cell];
  int v, t0, t1;
  if (ci >= 0) {
    v = tp.n_start + ci;
    t0 = tp.comb_inptr[ci];
    t1 = tp.comb_inptr[ci + 1];
  } else {
    const int f = -ci - 1;
    v = tp.n_pi + f;
    t0 = tp.A + f;
    t1 = t0 + 1;
  }
  float ax = gpin[2 * v], ay = gpin[2 * v + 1];
  for (int t = t0; t < t1; ++t) {
    ax += gpin[2 * (tp.M + t)];
    ay += gpin[2 * (tp.M + t) + 1];
  }
  gx[cell] += ax;
  gy[cell] += ay;
}

void wa_impl(tdp_graph g, const float *x, const float *y, float gamma, double *wl, float *gx, float *gy,
             hipStream_t s) {
  const Topo &tp = g->topo;
  prof_begin(g, TDP_STAGE_WA, s);
  constexpr int WB = RED_BLOCKS * 4, BB = 64;  // partial slots: chunked nets, then big nets
  // x == nullptr: the positions of the last timing update, whose cell
  // coordinates per slot it already gathered
  const float2 *xy = g->xy, *cxy = g->cxy_nm;
  if (x) {
    pack_xy(x, y, g->xy_wa, tp.N, s);
    xy = g->xy_wa;
    cxy = nullptr;
  }
  // (no launch for wide nets where the design has none)
  const int wb = std::min(WB, nb(tp.n_nm_chunks, 4)), bb = tp.n_big > 0 ? BB : 0;
  hipLaunchKernelGGL(k_wa_net, dim3(wb), dim3(256), 0, s, tp, xy, cxy, gamma, g->wa_gpin, g->red_wa);
  if (bb)
    hipLaunchKernelGGL(k_wa_big, dim3(bb), dim3(64), 0, s, tp, xy, gamma, g->wa_gpin, g->red_wa + wb);
  hipLaunchKernelGGL(k_sum_parts2, dim3(1), dim3(256), 0, s, wb + bb, g->red_wa, wl);
  hipLaunchKernelGGL(k_wa_cell, dim3(nb(tp.N, 256)), dim3(256), 0, s, tp, g->wa_gpin, gx, gy);
  prof_end(g, TDP_STAGE_WA, s);
}

template void stns_fwd_impl<float>(tdp_graph, const float *, const float *, float, double *, hipStream_t);
template void stns_fwd_impl<double>(tdp_graph, const float *, const float *, float, double *, hipStream_t);
template void stns_bwd_impl<float>(tdp_graph, const double *, float *, float *, hipStream_t);
template void stns_bwd_impl<double>(tdp_graph, const double *, float *, float *, hipStream_t);

}  // namespace tdp
