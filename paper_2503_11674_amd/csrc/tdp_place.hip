// The placement loop around the hot path: a bin-density penalty with its
// gradient, and one step of Nesterov's method (the paper's placer minimises
// wirelength + lambda * density (Eq. 1) + beta * PP (Eq. 6) with
// DREAMPlace's Nesterov optimiser; Sec. IV).
//
// Density: the die is cut into gx x gy bins of bw x bh, bin (i, j) at
// j * gx + i.  Cell c spreads its area a_c as a Gaussian centred on its
// position with standard deviations (bw, bh), integrated over each bin, over
// the (2R+1)^2 bins around the bin holding it (its indices clamped into the
// grid); mass the window puts off the die is reflected back in at the edges
// (mirror images, the Neumann boundary of an electrostatic density):
//   D(i, j) = sum_c a_c Wx_c(i) Wy_c(j),   Wx_c(i) = sum of Phi(upper) -
// Phi(lower) at the standardised edges of the window bins that fold onto i.  value = sum_b max(0, D_b - cap)^2 with
// cap = target * bw * bh, overflow = sum_b max(0, D_b - cap) / sum_c a_c.
//
// One evaluation: cells are sorted by bin (stable radix sort); each sorted
// cell writes its 2(2R+1) window weights (x weights times its area); each bin
// then gathers, in a fixed order, the weights of the cells in the bins whose
// windows reach it (a crowded bin with a whole workgroup); the gradient is a
// gather per cell over its window's overflow.  No floating-point atomics:
// results are bitwise reproducible.
// A cell's bin is decided in double precision (its position minus the
// grid origin, over the bin size), so that the decision does not depend on
// the rounding of a single-precision quotient.
#include "tdp_impl.h"
#include "tdp_look.h"
#include "tdp_prims.h"

namespace tdp {

static inline int nbk(long long n, int b) { return n > 0 ? (int)((n + b - 1) / b) : 1; }

constexpr int DN_BLOCK = 256;
constexpr int DN_PARTS = 1024;  // partial sums per reduction (fixed grid)
constexpr int DN_GROUPS = 256;  // the same where the last workgroup adds them up

__device__ __forceinline__ int dn_bin(float v, float v0, float w, int g, float &frac) {
  const double q = ((double)v - (double)v0) / (double)w;
  double f = floor(q);
  f = !(f >= 0.0) ? 0.0 : (f > (double)(g - 1) ? (double)(g - 1) : f);  // NaN -> bin 0: never out of the grid
  frac = (float)(q - f);  // position inside the bin in bin widths (outside [0, 1) when clamped)
  return (int)f;
}

// Phi(hi) - Phi(lo) for hi >= lo, from complementary error functions on the
// side where both are small (no cancellation between two values near 1)
__device__ __forceinline__ float gauss_mass(float lo, float hi) {
  const float s = 0.70710678118654752f;  // 1 / sqrt(2)
  if (lo >= 0.f) return 0.5f * (erfcf(lo * s) - erfcf(hi * s));
  if (hi <= 0.f) return 0.5f * (erfcf(-hi * s) - erfcf(-lo * s));
  return 1.f - 0.5f * (erfcf(hi * s) + erfcf(-lo * s));
}

__device__ __forceinline__ float gauss_pdf(float z) { return 0.39894228040143268f * expf(-0.5f * z * z); }

// Weight and its derivative (per unit of position) for grid bin i of a cell
// at fraction f of window bin b: the window bins u = b - R .. b + R that fold
// onto i (u itself inside the grid; u < 0 onto -1 - u, u >= g onto
// 2g - 1 - u, repeatedly), summed in window order.  Cells whose window lies
// inside the grid take the single direct term.
__device__ __forceinline__ void axis_weight(int b, float f, int g, int R, int i, float inv_w, float &wt,
                                            float &dt) {
  if (b - R >= 0 && b + R < g) {
    const float lo = (float)(i - b) - f, hi = lo + 1.f;
    wt = gauss_mass(lo, hi);
    dt = (gauss_pdf(lo) - gauss_pdf(hi)) * inv_w;
    return;
  }
  wt = 0.f;
  dt = 0.f;
  for (int k = 0; k <= 2 * R; ++k) {
    int v = b - R + k;
    for (int r = 0; r < 64 && (v < 0 || v >= g); ++r) v = v < 0 ? -1 - v : 2 * g - 1 - v;
    if (v != i) continue;
    const float lo = (float)(k - R) - f, hi = lo + 1.f;
    wt += gauss_mass(lo, hi);
    dt += (gauss_pdf(lo) - gauss_pdf(hi)) * inv_w;
  }
}

// Derivatives (per unit of position) of a cell's 2R+1 weights on one axis from
// the densities at the window bins' 2R+2 edges; weights (below) alike.  For
// windows inside the grid.
template <int R>
__device__ __forceinline__ void axis_slopes(float f, float inv_w, float (&dt)[2 * R + 1]) {
  float below = gauss_pdf((float)-R - f);
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    const float above = gauss_pdf((float)(k + 1 - R) - f);
    dt[k] = (below - above) * inv_w;
    below = above;
  }
}

// as gauss_mass between neighbouring edges, each edge's tail computed once
template <int R>
__device__ __forceinline__ void axis_masses(float f, float (&wt)[2 * R + 1]) {
  const float s = 0.70710678118654752f;  // 1 / sqrt(2)
  float lo = (float)-R - f;
  float tail = erfcf(fabsf(lo) * s);
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) {
    const float hi = (float)(k + 1 - R) - f;
    const float next = erfcf(fabsf(hi) * s);
    wt[k] = lo >= 0.f ? 0.5f * (tail - next) : (hi <= 0.f ? 0.5f * (next - tail) : 1.f - 0.5f * (next + tail));
    lo = hi;
    tail = next;
  }
}

__device__ __forceinline__ bool window_inside(int b, int g, int R) { return b - R >= 0 && b + R < g; }

// a cell's place in the sort: its id, and in the top bit whether it is fixed
constexpr uint32_t DN_FIXED = 0x80000000u;

__global__ void __launch_bounds__(DN_BLOCK) k_dn_keys(int n, const float *__restrict__ x, const float *__restrict__ y,
                                                       const uint8_t *__restrict__ fixed, DensityGrid gr,
                                                       uint32_t *__restrict__ key, uint32_t *__restrict__ val) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  float fx, fy;
  const int bx = dn_bin(x[c], gr.x0, gr.bw, gr.gx, fx);
  const int by = dn_bin(y[c], gr.y0, gr.bh, gr.gy, fy);
  key[c] = (uint32_t)by * (uint32_t)gr.gx + (uint32_t)bx;
  val[c] = (uint32_t)c | (fixed[c] ? DN_FIXED : 0u);
}

// start[b] = first sorted position with key >= b, for b in [0, G]: a binary
// search per bin (balanced however crowded the bins are).  No bin is listed as
// crowded yet.
__global__ void __launch_bounds__(DN_BLOCK) k_dn_starts(int n, int G, const uint32_t *__restrict__ key,
                                                         int32_t *__restrict__ start, int32_t *__restrict__ n_heavy) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b == 0) *n_heavy = 0;
  if (b > G) return;
  int lo = 0, hi = n;  // the answer lies in [lo, hi]
  while (lo < hi) {
    const int mid = lo + ((hi - lo) >> 1);
    if (key[mid] < (uint32_t)b) lo = mid + 1;
    else hi = mid;
  }
  start[b] = lo;
}

// Of sorted cell s, K = 2R + 1: its weights w[k * n + s] = a_c Wx(k - R) and
// w[(K + k) * n + s] = Wy(k - R), then its area and its fractions of a bin,
// for the gradient: what both need is gathered and evaluated once.  A thread
// per cell and axis (blockIdx.y).  Bound by the gathers and, on few cells, by
// the chain of error functions, 2R + 2 where the window lies inside the grid
// (4R + 2 in one thread for both axes: 39 us at 500,000 cells, R = 3; 25 now).
template <int R>
__global__ void __launch_bounds__(DN_BLOCK) k_dn_weights(int n, const uint32_t *__restrict__ order,
                                                          const float *__restrict__ x, const float *__restrict__ y,
                                                          const float *__restrict__ area, DensityGrid gr,
                                                          float *__restrict__ w) {
  constexpr int K = 2 * R + 1;
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  const bool is_y = blockIdx.y;
  if (s >= n) return;
  const int c = (int)(order[s] & ~DN_FIXED);
  const int g = is_y ? gr.gy : gr.gx;
  float f;
  const int b = dn_bin((is_y ? y : x)[c], is_y ? gr.y0 : gr.x0, is_y ? gr.bh : gr.bw, g, f);
  const float a = is_y ? 1.f : area[c];
  float wt[K];
  if (window_inside(b, g, R)) {
    axis_masses<R>(f, wt);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = b - R + k;
      float dt;
      wt[k] = 0.f;
      if (i >= 0 && i < g) axis_weight(b, f, g, R, i, 1.f, wt[k], dt);
    }
  }
  float *const mine = w + (is_y ? (size_t)K * n : 0) + s;
#pragma unroll
  for (int k = 0; k < K; ++k) mine[(size_t)k * n] = a * wt[k];
  float *const aux = w + (size_t)(2 * K) * n + s;
  if (!is_y) aux[0] = a;
  aux[(size_t)(is_y ? 2 : 1) * n] = f;
}

__device__ __forceinline__ void block_sum2(double &a, double &b) {
  __shared__ double sa[DN_BLOCK], sb[DN_BLOCK];
  sa[threadIdx.x] = a;
  sb[threadIdx.x] = b;
  __syncthreads();
  for (int o = DN_BLOCK / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sa[threadIdx.x] += sa[threadIdx.x + o];
      sb[threadIdx.x] += sb[threadIdx.x + o];
    }
    __syncthreads();
  }
  a = sa[0];
  b = sb[0];
}

// Bin gathers.  Keys are row-major (by * gx + bx), so the cells of the bins
// [i - R, i + R] of one row are one contiguous range of the sorted order: a
// bin's window is 2R+1 ranges.  A bin whose window holds at most DN_HEAVY
// cells sums each row's cells in sorted order, then the rows; a crowded bin is
// listed and summed by a whole workgroup (cells dealt to threads by position, a
// fixed-order tree over the threads).  Either way the sum depends on the data
// alone: results are bitwise reproducible.
constexpr int DN_HEAVY = 512;
constexpr int DN_LANES = 8;

__device__ __forceinline__ void window_row(const DensityGrid &gr, const int32_t *__restrict__ start, int i, int sj,
                                           int &s0, int &s1) {
  const int lo = sj * gr.gx + (i - gr.R > 0 ? i - gr.R : 0);
  const int hi = sj * gr.gx + (i + gr.R < gr.gx - 1 ? i + gr.R : gr.gx - 1);
  s0 = start[lo];
  s1 = start[hi + 1];
}

// the product a_c Wx_c(i) Wy_c(j) of sorted cell s in row sj = j - dj
__device__ __forceinline__ double dn_term(const DensityGrid &gr, const uint32_t *__restrict__ key,
                                          const float *__restrict__ w, int n, int K, int i, int sj, int dj, int s) {
  const int di = i - (int)(key[s] - (uint32_t)sj * (uint32_t)gr.gx);
  return (double)(w[(size_t)(di + gr.R) * n + s] * w[(size_t)(K + dj + gr.R) * n + s]);
}

// Workgroups go to the 8 XCDs in turn, each with an L2 of its own: consecutive
// `run` workgroups of bins (some rows of the grid) are given to one XCD, so
// that a row's weights are not read into all eight.
__device__ __forceinline__ int xcd_run(int blk, int nblk, int run) {
  const int round = blk / (8 * run), first = round * 8 * run;
  if (first + 8 * run > nblk) return blk;  // the ragged end keeps its order
  const int in = blk - first;
  return first + (in & 7) * run + (in >> 3);
}

// Radii up to DN_STRIP: 64 columns of bins by 16 - 2R rows per workgroup.  Wave
// q takes source row q of the strip's window and lane i its cells about column
// i: one x weight and 2R+1 y weights per cell give the cell's terms for all
// 2R+1 bins of the column, kept in registers; the bins then add up their
// rows' parts from LDS.  The lanes of a wave read one row's cells, so a load
// touches a few lines.  500,000 cells in 512 x 512 bins, R = 3: 59 us; eight
// lanes a bin, a row each, took 105, a thread a bin 222.
constexpr int DN_STRIP = 4;
// A row with more cells than this makes its bins crowded: a lane's cells are a
// serial chain, and one of 500 in a strip (cells against the die's edge) took
// twice as long as all the rest (146 us against 59 and 8 more in k_dn_heavy).
constexpr int DN_ROW = 64;
// On a grid of many bins whose rows hold almost that many cells on average, that
// would make crowded bins of a good part of them, each with a workgroup's fixed
// cost: there a row may have some more.  500,000 cells evenly over 200 x 200 bins,
// R = 2 (rows of 62), the whole evaluation: 215 us against 258 (222 with a thread a
// bin); 256 x 256, R = 3 (53): 211 against 260.  On 128 x 128, R = 1 (91) or where
// the cells are few for the bins, the lower bound is the better one (165 against
// 177, clusters 250 against 239).
constexpr int DN_ROW_FULL = 80, DN_FULL_MEAN = 40, DN_FULL_BINS = 1 << 15;

template <int R>
__global__ void __launch_bounds__(1024) k_dn_strip(int n, int run, int row, DensityGrid gr, const int32_t *__restrict__ start,
                                                    const float *__restrict__ w, float *__restrict__ map,
                                                    int32_t *__restrict__ heavy, int32_t *__restrict__ n_heavy) {
  constexpr int K = 2 * R + 1, ROWS = 16, H = ROWS - 2 * R;
  __shared__ double s_part[ROWS][K][64];
  __shared__ int s_cnt[ROWS][64];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int cols = (gr.gx + 63) / 64, blk = xcd_run(blockIdx.x, gridDim.x, run);
  const int i = (blk % cols) * 64 + lane, j0 = (blk / cols) * H;
  const int sj = j0 - R + q;  // the wave's source row
  double d[K];
#pragma unroll
  for (int k = 0; k < K; ++k) d[k] = 0.0;
  int cnt = 0;
  if (i < gr.gx && sj >= 0 && sj < gr.gy) {
    // first cells of the row's window bins; bins past the grid's edge are empty
    int at[K + 1];
#pragma unroll
    for (int k = 0; k <= K; ++k) at[k] = start[sj * gr.gx + min(max(i - R + k, 0), gr.gx)];
    cnt = at[K] - at[0];
    if (cnt <= row) {  // (otherwise every bin that needs the row is crowded)
#pragma unroll 2
      for (int s = at[0]; s < at[K]; ++s) {
        int col = 2 * R;  // the x weight of a cell k bins along is its (2R - k)-th
#pragma unroll
        for (int k = 1; k < K; ++k) col -= s >= at[k];
        const float wx = w[(size_t)col * n + s];
#pragma unroll
        for (int k = 0; k < K; ++k) d[k] += (double)(wx * w[(size_t)(K + k) * n + s]);
      }
    }
  }
  s_cnt[q][lane] = cnt;
#pragma unroll
  for (int k = 0; k < K; ++k) s_part[q][k][lane] = d[k];
  __syncthreads();
  // bin row q of the strip: source row q + r holds its part at offset dj = R - r
  if (q >= H || j0 + q >= gr.gy || i >= gr.gx) return;
  int most = 0;
  cnt = 0;
  double sum = 0.0;
#pragma unroll
  for (int r = 2 * R; r >= 0; --r) {
    cnt += s_cnt[q + r][lane];
    most = max(most, s_cnt[q + r][lane]);
    sum += s_part[q + r][2 * R - r][lane];
  }
  const int b = (j0 + q) * gr.gx + i;
  if (cnt > DN_HEAVY || most > row) heavy[atomicAdd(n_heavy, 1)] = b;  // summed by k_dn_heavy
  else map[b] = (float)sum;
}

// wider windows (a strip's parts would not fit LDS): DN_LANES threads per bin, a
// thread the rows lane, lane + DN_LANES, ...
template <int R>
__global__ void __launch_bounds__(DN_BLOCK) k_dn_bins(int n, int run, DensityGrid gr, const int32_t *__restrict__ start,
                                                       const float *__restrict__ w, float *__restrict__ map,
                                                       int32_t *__restrict__ heavy, int32_t *__restrict__ n_heavy) {
  constexpr int K = 2 * R + 1;
  const int G = gr.gx * gr.gy;
  const int lane = threadIdx.x & (DN_LANES - 1);
  const int b = xcd_run(blockIdx.x, gridDim.x, run) * (DN_BLOCK / DN_LANES) + threadIdx.x / DN_LANES;
  const int i = b % gr.gx, j = b / gr.gx;
  int cnt = 0;
  if (b < G) {
    for (int dj = lane - R; dj <= R; dj += DN_LANES) {
      const int sj = j - dj;
      if (sj < 0 || sj >= gr.gy) continue;
      int s0, s1;
      window_row(gr, start, i, sj, s0, s1);
      cnt += s1 - s0;
    }
  }
#pragma unroll
  for (int o = 1; o < DN_LANES; o <<= 1) cnt += __shfl_xor(cnt, o, DN_LANES);
  double d = 0.0;
  if (b < G && cnt <= DN_HEAVY) {
    for (int dj = lane - R; dj <= R; dj += DN_LANES) {
      const int sj = j - dj;
      if (sj < 0 || sj >= gr.gy) continue;
      // first cells of the row's window bins; bins past the grid's edge are empty
      int at[K + 1];
#pragma unroll
      for (int k = 0; k <= K; ++k) at[k] = start[sj * gr.gx + min(max(i - R + k, 0), gr.gx)];
      const float *wy = w + (size_t)(K + dj + R) * n;
#pragma unroll 4
      for (int s = at[0]; s < at[K]; ++s) {
        int col = 2 * R;  // the x weight of a cell k bins along is its (2R - k)-th
#pragma unroll
        for (int k = 1; k < K; ++k) col -= s >= at[k];
        d += (double)(w[(size_t)col * n + s] * wy[s]);
      }
    }
  }
#pragma unroll
  for (int o = 1; o < DN_LANES; o <<= 1) d += __shfl_xor(d, o, DN_LANES);
  if (b >= G || lane != 0) return;
  if (cnt > DN_HEAVY) heavy[atomicAdd(n_heavy, 1)] = b;  // summed by k_dn_heavy
  else map[b] = (float)d;
}

// one workgroup per listed bin (grid-stride over the list), a wave a row of
// its window
constexpr int DN_WAVES = 8;

__global__ void __launch_bounds__(64 * DN_WAVES) k_dn_heavy(int n, DensityGrid gr, const int32_t *__restrict__ start,
                                                            const uint32_t *__restrict__ key,
                                                            const float *__restrict__ w,
                                                            const int32_t *__restrict__ heavy,
                                                            const int32_t *__restrict__ n_heavy,
                                                            float *__restrict__ map) {
  __shared__ double s_row[2][DN_WAVES];
  const int R = gr.R, K = 2 * R + 1, lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int nh = *n_heavy;
  int odd = 0;
  for (int h = blockIdx.x; h < nh; h += gridDim.x, odd ^= 1) {
    const int b = heavy[h];
    const int i = b % gr.gx, j = b / gr.gx;
    double d = 0.0;
    for (int dj = q - R; dj <= R; dj += DN_WAVES) {
      const int sj = j - dj;
      if (sj < 0 || sj >= gr.gy) continue;
      int s0, s1;
      window_row(gr, start, i, sj, s0, s1);
#pragma unroll 4
      for (int s = s0 + lane; s < s1; s += 64) d += dn_term(gr, key, w, n, K, i, sj, dj, s);
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) d += __shfl_xor(d, o, 64);
    if (lane == 0) s_row[odd][q] = d;
    __syncthreads();  // (the other half of s_row is this bin's successor's)
    if (threadIdx.x == 0) {
      d = 0.0;
#pragma unroll
      for (int r = 0; r < DN_WAVES; ++r) d += s_row[odd][r];
      map[b] = (float)d;
    }
  }
}

// sums of o^2 and o over the finished map, o = max(0, D - cap): a part per
// workgroup, added up by the last one
__global__ void __launch_bounds__(DN_BLOCK) k_dn_reduce(DensityGrid gr, const float *__restrict__ map,
                                                         double *__restrict__ part, uint32_t *__restrict__ ctr,
                                                         double inv_area, double *value, double *overflow) {
  const uint32_t launch = ctr[0];
  const int G = gr.gx * gr.gy;
  const float cap = gr.target * gr.bw * gr.bh;
  double so2 = 0.0, so = 0.0;
  for (int b = blockIdx.x * DN_BLOCK + threadIdx.x; b < G; b += gridDim.x * DN_BLOCK) {
    const float df = map[b];
    const double o = df > cap ? (double)df - (double)cap : 0.0;
    so2 += o * o;
    so += o;
  }
  block_sum2(so2, so);
  if (threadIdx.x == 0) {
    pub_st(part + blockIdx.x, so2);
    pub_st(part + DN_PARTS + blockIdx.x, so);
  }
  if (!look_done(Look{nullptr, ctr, nullptr}, launch)) return;
  so2 = so = 0.0;
  for (int i = threadIdx.x; i < (int)gridDim.x; i += DN_BLOCK) {
    so2 += pub_ld(part + i);
    so += pub_ld(part + DN_PARTS + i);
  }
  block_sum2(so2, so);
  if (threadIdx.x == 0) {
    if (value) *value = so2;
    if (overflow) *overflow = so * inv_area;
  }
}

// gradient of the penalty on movable cells: += scale * d value / d (x, y).
//   d/dx = 2 a sum_j Wy(j) sum_i Wx'(i) o(i, j),  d/dy likewise.
// Threads take the cells in bin order, so that a wave's windows overlap and
// share the map's cache lines; weights, areas and fractions come from
// k_dn_weights in that order, so only the gradient itself is gathered.  The
// window is in registers (R is a template parameter).  500,000 cells, R = 3:
// 47 us; with positions, areas and error functions once more, 62.
template <int R>
__global__ void __launch_bounds__(DN_BLOCK) k_dn_grad(int n, const uint32_t *__restrict__ order,
                                                       const uint32_t *__restrict__ key, const float *__restrict__ w,
                                                       DensityGrid gr, const float *__restrict__ map, float scale,
                                                       float *__restrict__ gx, float *__restrict__ gy) {
  constexpr int K = 2 * R + 1;
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const uint32_t oc = order[s];
  if (oc & DN_FIXED) return;
  const int c = (int)oc, bin = (int)key[s];
  const int by = bin / gr.gx, bx = bin - by * gr.gx;
  const float a = w[(size_t)(2 * K) * n + s], fx = w[(size_t)(2 * K + 1) * n + s], fy = w[(size_t)(2 * K + 2) * n + s];
  const float cap = gr.target * gr.bw * gr.bh;
  float wx[K], dx[K], wy[K], dy[K];  // (wx times the area)
#pragma unroll
  for (int k = 0; k < K; ++k) {
    wx[k] = w[(size_t)k * n + s];
    wy[k] = w[(size_t)(K + k) * n + s];
  }
  if (window_inside(bx, gr.gx, R)) {
    axis_slopes<R>(fx, 1.f / gr.bw, dx);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int i = bx - R + k;
      float wt;
      dx[k] = 0.f;
      if (i >= 0 && i < gr.gx) axis_weight(bx, fx, gr.gx, R, i, 1.f / gr.bw, wt, dx[k]);
    }
  }
  if (window_inside(by, gr.gy, R)) {
    axis_slopes<R>(fy, 1.f / gr.bh, dy);
  } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int j = by - R + k;
      float wt;
      dy[k] = 0.f;
      if (j >= 0 && j < gr.gy) axis_weight(by, fy, gr.gy, R, j, 1.f / gr.bh, wt, dy[k]);
    }
  }
  float ax = 0.f, ay = 0.f;
#pragma unroll
  for (int kj = 0; kj < K; ++kj) {
    const int j = by - R + kj;
    if (j < 0 || j >= gr.gy) continue;
    float sx = 0.f, sy = 0.f;
#pragma unroll
    for (int ki = 0; ki < K; ++ki) {
      const int i = bx - R + ki;
      if (i < 0 || i >= gr.gx) continue;
      const float o = map[j * gr.gx + i] - cap;
      if (o <= 0.f) continue;
      sx += o * dx[ki];
      sy += o * wx[ki];
    }
    ax += sx * wy[kj];
    ay += sy * dy[kj];
  }
  gx[c] += 2.f * a * scale * ax;
  gy[c] += 2.f * scale * ay;
}

template <int R>
static void density_launch(tdp_graph g, const float *x, const float *y, float scale, double *value, double *overflow,
                           float *gx, float *gy, float *map_out, hipStream_t s) {
  const int n = g->topo.N;
  const DensityGrid &gr = g->dn;
  const int G = gr.gx * gr.gy;
  Sorted<uint32_t> so{g->dn_k0, g->dn_v0};
  if (n > 0) {
    hipLaunchKernelGGL(k_dn_keys, dim3(nbk(n, DN_BLOCK)), dim3(DN_BLOCK), 0, s, n, x, y, g->topo.cell_fixed, gr,
                       g->dn_k0, g->dn_v0);
    so = radix_sort(g->dn_k0, g->dn_v0, g->dn_k1, g->dn_v1, n, nullptr, g->dn_key_bits, 11, g->dn_hist, s);
    hipLaunchKernelGGL(k_dn_weights<R>, dim3(nbk(n, DN_BLOCK), 2), dim3(DN_BLOCK), 0, s, n, (const uint32_t *)so.vals,
                       x, y, (const float *)g->dn_area, gr, g->dn_w);
  }
  hipLaunchKernelGGL(k_dn_starts, dim3(nbk((long long)G + 1, DN_BLOCK)), dim3(DN_BLOCK), 0, s, n, G,
                     (const uint32_t *)so.keys, g->dn_start, g->dn_nheavy);
  float *map = map_out ? map_out : g->dn_map;
  if constexpr (R <= DN_STRIP) {
    const int cols = nbk(gr.gx, 64);
    const bool full = G >= DN_FULL_BINS && (long long)n * (2 * R + 1) > (long long)DN_FULL_MEAN * G;
    const int row = full ? DN_ROW_FULL : DN_ROW;
    hipLaunchKernelGGL(k_dn_strip<R>, dim3(cols * nbk(gr.gy, 16 - 2 * R)), dim3(1024), 0, s, n, 2 * cols, row, gr,
                       (const int32_t *)g->dn_start, (const float *)g->dn_w, map, g->dn_heavy, g->dn_nheavy);
  } else {
    hipLaunchKernelGGL(k_dn_bins<R>, dim3(nbk(G, DN_BLOCK / DN_LANES)), dim3(DN_BLOCK), 0, s, n,
                       8 * nbk(gr.gx, DN_BLOCK / DN_LANES), gr, (const int32_t *)g->dn_start, (const float *)g->dn_w,
                       map, g->dn_heavy, g->dn_nheavy);
  }
  hipLaunchKernelGGL(k_dn_heavy, dim3(DN_PARTS), dim3(64 * DN_WAVES), 0, s, n, gr, (const int32_t *)g->dn_start,
                     (const uint32_t *)so.keys, (const float *)g->dn_w, (const int32_t *)g->dn_heavy,
                     (const int32_t *)g->dn_nheavy, map);
  hipLaunchKernelGGL(k_dn_reduce, dim3(std::min(DN_GROUPS, nbk(G, DN_BLOCK))), dim3(DN_BLOCK), 0, s, gr,
                     (const float *)map, g->dn_part, g->dn_ctr, g->dn_total_area > 0 ? 1.0 / g->dn_total_area : 0.0,
                     value, overflow);
  // (so.vals and so.keys: this call's sort)
  if (gx && gy && n > 0)
    hipLaunchKernelGGL(k_dn_grad<R>, dim3(nbk(n, DN_BLOCK)), dim3(DN_BLOCK), 0, s, n, (const uint32_t *)so.vals,
                       (const uint32_t *)so.keys, (const float *)g->dn_w, gr, (const float *)map, scale, gx, gy);
}

void density_impl(tdp_graph g, const float *x, const float *y, float scale, double *value, double *overflow,
                  float *gx, float *gy, float *map_out, hipStream_t s) {
  prof_begin(g, TDP_STAGE_DENSITY, s);
  switch (g->dn.R) {
    case 0: density_launch<0>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 1: density_launch<1>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 2: density_launch<2>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 3: density_launch<3>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 4: density_launch<4>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 5: density_launch<5>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 6: density_launch<6>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    case 7: density_launch<7>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
    default: density_launch<8>(g, x, y, scale, value, overflow, gx, gy, map_out, s); break;
  }
  prof_end(g, TDP_STAGE_DENSITY, s);
}

// ---------------------------------------------------------------- Nesterov
// One step on the 2n coordinates of the graph's cells (frozen: fixed cells):
//   q = gradient / max(1, pdiv_c);  alpha = |v - vp| / |q - gp| (alpha0 on
//   the first step or when that is not a positive number);
//   u' = clamp(v - alpha q);  v' = clamp(u' + coef (u' - u));
//   then vp = v, gp = q, u = u', v = v'.
__global__ void __launch_bounds__(DN_BLOCK) k_nest_norms(int n, const uint8_t *__restrict__ fixed,
                                                          const float *__restrict__ pdiv, const float *__restrict__ gx,
                                                          const float *__restrict__ gy, const float *__restrict__ vx,
                                                          const float *__restrict__ vy, const float *__restrict__ vpx,
                                                          const float *__restrict__ vpy, const float *__restrict__ gpx,
                                                          const float *__restrict__ gpy, double *__restrict__ part) {
  double dv = 0.0, dg = 0.0;
  for (int c = blockIdx.x * DN_BLOCK + threadIdx.x; c < n; c += DN_PARTS * DN_BLOCK) {
    if (fixed[c]) continue;
    const float p = pdiv[c] > 1.f ? pdiv[c] : 1.f;
    const double ex = (double)vx[c] - (double)vpx[c], ey = (double)vy[c] - (double)vpy[c];
    const double qx = (double)(gx[c] / p) - (double)gpx[c], qy = (double)(gy[c] / p) - (double)gpy[c];
    dv += ex * ex + ey * ey;
    dg += qx * qx + qy * qy;
  }
  block_sum2(dv, dg);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = dv;
    part[DN_PARTS + blockIdx.x] = dg;
  }
}

__global__ void __launch_bounds__(DN_BLOCK) k_nest_alpha(const double *__restrict__ part, double alpha0, int first,
                                                          double *__restrict__ alpha) {
  double dv = 0.0, dg = 0.0;
  for (int i = threadIdx.x; i < DN_PARTS; i += DN_BLOCK) {
    dv += part[i];
    dg += part[DN_PARTS + i];
  }
  block_sum2(dv, dg);
  if (threadIdx.x == 0) {
    double a = alpha0;
    if (!first && dg > 0.0) {
      const double r = sqrt(dv) / sqrt(dg);
      if (r > 0.0 && isfinite(r)) a = r;
    }
    *alpha = a;
  }
}

__global__ void __launch_bounds__(DN_BLOCK) k_nest_update(int n, const uint8_t *__restrict__ fixed,
                                                           const float *__restrict__ pdiv, const float *__restrict__ gx,
                                                           const float *__restrict__ gy, float *__restrict__ vx,
                                                           float *__restrict__ vy, float *__restrict__ ux,
                                                           float *__restrict__ uy, float *__restrict__ vpx,
                                                           float *__restrict__ vpy, float *__restrict__ gpx,
                                                           float *__restrict__ gpy, float coef,
                                                           const double *__restrict__ alpha, float xlo, float xhi,
                                                           float ylo, float yhi) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= n) return;
  const float x = vx[c], yv = vy[c];
  if (fixed[c]) {
    vpx[c] = x;
    vpy[c] = yv;
    gpx[c] = 0.f;
    gpy[c] = 0.f;
    return;
  }
  const float p = pdiv[c] > 1.f ? pdiv[c] : 1.f;
  const float qx = gx[c] / p, qy = gy[c] / p;
  const float a = (float)*alpha;
  const float nux = fminf(fmaxf(x - a * qx, xlo), xhi), nuy = fminf(fmaxf(yv - a * qy, ylo), yhi);
  const float nvx = fminf(fmaxf(nux + coef * (nux - ux[c]), xlo), xhi);
  const float nvy = fminf(fmaxf(nuy + coef * (nuy - uy[c]), ylo), yhi);
  vpx[c] = x;
  vpy[c] = yv;
  gpx[c] = qx;
  gpy[c] = qy;
  ux[c] = nux;
  uy[c] = nuy;
  vx[c] = nvx;
  vy[c] = nvy;
}

void nesterov_impl(tdp_graph g, const float *gx, const float *gy, const float *pdiv, float *vx, float *vy, float *ux,
                   float *uy, float *vpx, float *vpy, float *gpx, float *gpy, double coef, double alpha0, int first,
                   float xlo, float xhi, float ylo, float yhi, double *alpha_out, hipStream_t s) {
  const int n = g->topo.N;
  const uint8_t *fixed = g->topo.cell_fixed;
  double *alpha = alpha_out ? alpha_out : g->nest_alpha;
  hipLaunchKernelGGL(k_nest_norms, dim3(DN_PARTS), dim3(DN_BLOCK), 0, s, n, fixed, pdiv, gx, gy,
                     (const float *)vx, (const float *)vy, (const float *)vpx, (const float *)vpy,
                     (const float *)gpx, (const float *)gpy, g->nest_part);
  hipLaunchKernelGGL(k_nest_alpha, dim3(1), dim3(DN_BLOCK), 0, s, (const double *)g->nest_part, alpha0, first, alpha);
  if (n > 0)
    hipLaunchKernelGGL(k_nest_update, dim3(nbk(n, DN_BLOCK)), dim3(DN_BLOCK), 0, s, n, fixed, pdiv, gx, gy, vx, vy, ux,
                       uy, vpx, vpy, gpx, gpy, (float)coef, (const double *)alpha, xlo, xhi, ylo, yhi);
}

// sum over cells of |a_c| + |b_c| (an L1 norm of a gradient), fixed order
__global__ void __launch_bounds__(DN_BLOCK) k_abs_parts(int n, const float *__restrict__ a,
                                                         const float *__restrict__ b, double *__restrict__ part) {
  double s = 0.0, unused = 0.0;
  for (int c = blockIdx.x * DN_BLOCK + threadIdx.x; c < n; c += DN_PARTS * DN_BLOCK)
    s += (double)fabsf(a[c]) + (double)fabsf(b[c]);
  block_sum2(s, unused);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

__global__ void __launch_bounds__(DN_BLOCK) k_abs_final(const double *__restrict__ part, double *out) {
  double s = 0.0, unused = 0.0;
  for (int i = threadIdx.x; i < DN_PARTS; i += DN_BLOCK) s += part[i];
  block_sum2(s, unused);
  if (threadIdx.x == 0) *out = s;
}

void abs_sum_impl(tdp_graph g, const float *a, const float *b, double *out, hipStream_t s) {
  hipLaunchKernelGGL(k_abs_parts, dim3(DN_PARTS), dim3(DN_BLOCK), 0, s, g->topo.N, a, b, g->nest_part);
  hipLaunchKernelGGL(k_abs_final, dim3(1), dim3(DN_BLOCK), 0, s, (const double *)g->nest_part, out);
}

int density_parts() { return DN_PARTS; }

}  // namespace tdp
