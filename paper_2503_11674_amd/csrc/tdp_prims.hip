// Device primitives: exclusive scan and a stable LSD radix sort.
//
// Both take a host capacity `cap` (sizes the grid) and an optional device
// count `d_n` (the live length, read on the device) so that callers never
// have to read a count back to the host; this keeps every call capturable in
// a hipGraph.  Results are deterministic: no floating-point atomics, integer
// counts only.
#include "tdp_prims.h"

#include "tdp_look.h"

namespace tdp {

constexpr int SCAN_BLOCK = 256;
constexpr int SCAN_ITEMS = 16;  // four int4 per thread
constexpr int SCAN_TILE = SCAN_BLOCK * SCAN_ITEMS;

// a thread's SCAN_ITEMS consecutive values starting at base (16-byte
// aligned): vector loads for a full run, element loads in the ragged tail
__device__ __forceinline__ void load_items(const int32_t *in, int base, int n, int (&v)[SCAN_ITEMS]) {
  if (base + SCAN_ITEMS <= n) {
    const int4 *p = (const int4 *)(in + base);
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS / 4; ++q) {
      const int4 x = p[q];
      v[4 * q] = x.x;
      v[4 * q + 1] = x.y;
      v[4 * q + 2] = x.z;
      v[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) v[i] = base + i < n ? in[base + i] : 0;
  }
}

__device__ __forceinline__ void store_items(int32_t *out, int base, int n, const int (&v)[SCAN_ITEMS]) {
  if (base + SCAN_ITEMS <= n) {
    int4 *p = (int4 *)(out + base);
#pragma unroll
    for (int q = 0; q < SCAN_ITEMS / 4; ++q) p[q] = make_int4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i)
      if (base + i < n) out[base + i] = v[i];
  }
}

__device__ __forceinline__ int live_count(int cap, const int32_t *d_n) {
  if (!d_n) return cap;
  int n = *d_n;
  return n < cap ? (n < 0 ? 0 : n) : cap;
}

// inclusive scan of one value per thread across a 256-thread block
__device__ __forceinline__ int block_inclusive_scan(int v, int *sh /*[4]*/) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63) sh[wid] = v;
  __syncthreads();
  int add = 0;
  for (int w = 0; w < wid; ++w) add += sh[w];
  __syncthreads();
  return v + add;
}

__global__ void __launch_bounds__(SCAN_BLOCK) k_scan_reduce(const int32_t *__restrict__ in, int cap,
                                                             const int32_t *d_n, int32_t *__restrict__ part) {
  __shared__ int sh[4];
  const int n = live_count(cap, d_n);
  const int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  int v[SCAN_ITEMS];
  load_items(in, base, n, v);
  int s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) s += v[i];
  int incl = block_inclusive_scan(s, sh);
  if (threadIdx.x == SCAN_BLOCK - 1) part[blockIdx.x] = incl;
}

// one block: exclusive scan of the per-tile sums in place, total to *d_total
__global__ void __launch_bounds__(SCAN_BLOCK) k_scan_partials(int32_t *__restrict__ part, int nparts,
                                                               int32_t *d_total) {
  __shared__ int sh[4];
  __shared__ int block_total;
  int carry = 0;
  for (int b0 = 0; b0 < nparts; b0 += SCAN_BLOCK) {
    int i = b0 + threadIdx.x;
    int v = i < nparts ? part[i] : 0;
    int incl = block_inclusive_scan(v, sh);
    if (i < nparts) part[i] = carry + incl - v;
    if (threadIdx.x == SCAN_BLOCK - 1) block_total = incl;
    __syncthreads();
    carry += block_total;
    __syncthreads();
  }
  if (threadIdx.x == 0 && d_total) *d_total = carry;
}

// (in and out may be the same array: a thread reads its items before it
// writes them and no other thread touches them)
__global__ void __launch_bounds__(SCAN_BLOCK) k_scan_down(const int32_t *in, int cap, const int32_t *d_n,
                                                           const int32_t *__restrict__ part, int32_t *out) {
  __shared__ int sh[4];
  const int n = live_count(cap, d_n);
  const int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  int v[SCAN_ITEMS];
  load_items(in, base, n, v);
  int s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) s += v[i];
  int incl = block_inclusive_scan(s, sh);
  int run = part[blockIdx.x] + incl - s;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int x = v[i];
    v[i] = run;
    run += x;
  }
  store_items(out, base, n, v);
}

// Second pass without a separate scan of the tile sums: every tile adds up
// the sums of the tiles before it itself (a few thousand integers from L2),
// which saves a launch; the last live tile writes the total.
__global__ void __launch_bounds__(SCAN_BLOCK) k_scan_down_sum(const int32_t *in, int cap, const int32_t *d_n,
                                                               const int32_t *__restrict__ part, int32_t *out,
                                                               int32_t *d_total) {
  __shared__ int sh[4];
  __shared__ int offset;
  const int n = live_count(cap, d_n);
  const int tiles = n > 0 ? (n + SCAN_TILE - 1) / SCAN_TILE : 1;
  if ((int)blockIdx.x >= tiles) return;
  int acc = 0;
  for (int i = threadIdx.x; i < (int)blockIdx.x; i += SCAN_BLOCK) acc += part[i];
  acc = block_inclusive_scan(acc, sh);
  if (threadIdx.x == SCAN_BLOCK - 1) offset = acc;
  __syncthreads();
  const int base = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_ITEMS;
  int v[SCAN_ITEMS];
  load_items(in, base, n, v);
  int s = 0;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) s += v[i];
  const int incl = block_inclusive_scan(s, sh);
  int run = offset + incl - s;
#pragma unroll
  for (int i = 0; i < SCAN_ITEMS; ++i) {
    const int x = v[i];
    v[i] = run;
    run += x;
  }
  store_items(out, base, n, v);
  if (d_total && (int)blockIdx.x == tiles - 1 && threadIdx.x == SCAN_BLOCK - 1) *d_total = offset + incl;
}

int scan_tmp_size(int cap) { return (cap + SCAN_TILE - 1) / SCAN_TILE + 1; }

void scan_exclusive(const int32_t *in, int32_t *out, int cap, const int32_t *d_n, int32_t *d_total,
                    int32_t *tmp, hipStream_t s) {
  if (cap <= 0) {
    hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(SCAN_BLOCK), 0, s, tmp, 0, d_total);
    return;
  }
  int nb = (cap + SCAN_TILE - 1) / SCAN_TILE;
  hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(SCAN_BLOCK), 0, s, in, cap, d_n, tmp);
  if (nb <= 8192) {
    hipLaunchKernelGGL(k_scan_down_sum, dim3(nb), dim3(SCAN_BLOCK), 0, s, in, cap, d_n, tmp, out, d_total);
    return;
  }
  hipLaunchKernelGGL(k_scan_partials, dim3(1), dim3(SCAN_BLOCK), 0, s, tmp, nb, d_total);
  hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(SCAN_BLOCK), 0, s, in, cap, d_n, tmp, out);
}

// ------------------------------------------------------------------ sort
// Tiles of 4,096 keys, digits of up to 11 bits: 32-bit keys take three passes.
// A pass is a histogram per tile and a scatter.  The scatter's workgroups add
// up the tiles' histograms themselves while there are few (RS_DIRECT); beyond
// that a launch between the two turns them into sums down the tiles.  Within a
// tile every wave ranks its own 512 keys against its own counters, so a tile
// needs a handful of barriers, not three per 256 keys.  500,000 keys of 18 bits:
// 48 us in 6 launches, against 66 in 12 with 8-bit digits, a scan of the
// histograms per pass and 2,048-key tiles.
constexpr int RS_BLOCK = 512;
constexpr int RS_WAVES = RS_BLOCK / 64;
constexpr int RS_ITEMS = 8;
constexpr int RS_TILE = RS_BLOCK * RS_ITEMS;
constexpr int RS_MAX_DIGIT = 11;
constexpr int RS_DIRECT = 64;  // tiles

template <typename Key>
__device__ __forceinline__ uint32_t digit_of(Key k, int shift, int width) {
  return (uint32_t)(k >> shift) & ((1u << width) - 1);
}

// hist[tile][digit]
template <typename Key>
__global__ void __launch_bounds__(RS_BLOCK) k_rs_hist(const Key *__restrict__ keys, int cap, const int32_t *d_n,
                                                       int shift, int width, int32_t *__restrict__ hist) {
  __shared__ int cnt[1 << RS_MAX_DIGIT];
  const int n = live_count(cap, d_n);
  const int ntiles = (n + RS_TILE - 1) / RS_TILE;
  if ((int)blockIdx.x >= ntiles) return;
  const int R = 1 << width;
  for (int d = threadIdx.x; d < R; d += RS_BLOCK) cnt[d] = 0;
  __syncthreads();
  const int base = blockIdx.x * RS_TILE;
  // every key of the thread is requested before the first count
  uint32_t dg[RS_ITEMS];
#pragma unroll
  for (int j = 0; j < RS_ITEMS; ++j) {
    const int i = base + j * RS_BLOCK + threadIdx.x;
    dg[j] = i < n ? digit_of(keys[i], shift, width) : ~0u;
  }
#pragma unroll
  for (int j = 0; j < RS_ITEMS; ++j)
    if (dg[j] != ~0u) atomicAdd(&cnt[dg[j]], 1);
  __syncthreads();
  for (int d = threadIdx.x; d < R; d += RS_BLOCK) hist[(size_t)blockIdx.x * R + d] = cnt[d];
}

// many tiles: hist becomes the sum over the tiles before, tot[digit] over all.
// 64 digits per workgroup, 16 runs of tiles each
__global__ void __launch_bounds__(1024) k_rs_cols(int cap, const int32_t *d_n, int width, int32_t *__restrict__ hist,
                                                   int32_t *__restrict__ tot) {
  __shared__ int s_run[16][64];
  const int n = live_count(cap, d_n);
  const int ntiles = (n + RS_TILE - 1) / RS_TILE;
  if (ntiles <= RS_DIRECT) return;
  const int R = 1 << width;
  const int d = blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6;
  const bool on = d < R;
  const int per = (ntiles + 15) / 16, t0 = min(g * per, ntiles), t1 = min(t0 + per, ntiles);
  int sum = 0;
  if (on) {
#pragma unroll 8
    for (int t = t0; t < t1; ++t) sum += hist[(size_t)t * R + d];
  }
  s_run[g][threadIdx.x & 63] = sum;
  __syncthreads();
  int run = 0;
  for (int q = 0; q < g; ++q) run += s_run[q][threadIdx.x & 63];
  if (!on) return;
  for (int t = t0; t < t1; t += 8) {
    int h[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) h[q] = t + q < t1 ? hist[(size_t)(t + q) * R + d] : 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (t + q < t1) hist[(size_t)(t + q) * R + d] = run;
      run += h[q];
    }
  }
  if (g == 15) tot[d] = run;
}

template <typename Key>
__global__ void __launch_bounds__(RS_BLOCK) k_rs_scatter(const Key *__restrict__ kin,
                                                          const uint32_t *__restrict__ vin, int cap,
                                                          const int32_t *d_n, int shift, int width,
                                                          const int32_t *__restrict__ hist,
                                                          const int32_t *__restrict__ tot, Key *__restrict__ kout,
                                                          uint32_t *__restrict__ vout) {
  __shared__ __align__(16) uint16_t wcnt[RS_WAVES][1 << RS_MAX_DIGIT];  // keys of the wave seen with a digit
  __shared__ int base[1 << RS_MAX_DIGIT];                               // the tile's first place for a digit
  const int n = live_count(cap, d_n);
  const int ntiles = (n + RS_TILE - 1) / RS_TILE;
  const int tile = blockIdx.x;
  if (tile >= ntiles) return;
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int R = 1 << width;
  // every key and value of the thread is requested before the ranking: wave w
  // takes the w-th 512 of the tile, in rounds of 64
  const int i0 = tile * RS_TILE + wid * (RS_TILE / RS_WAVES) + lane;
  Key kk[RS_ITEMS];
  uint32_t vv[RS_ITEMS];
#pragma unroll
  for (int j = 0; j < RS_ITEMS; ++j) {
    const int i = i0 + j * 64;
    kk[j] = i < n ? kin[i] : (Key)0;
    vv[j] = i < n ? vin[i] : 0u;
  }
  uint4 *z = (uint4 *)&wcnt[0][0];
  for (int q = tid; q < (int)(sizeof wcnt / 16); q += RS_BLOCK) z[q] = make_uint4(0, 0, 0, 0);
  // the tile's first place for each digit: the keys of smaller digits, then
  // those of this digit in the tiles before
  constexpr int PER = (1 << RS_MAX_DIGIT) / RS_BLOCK;  // digits per thread, consecutive
  int before[PER], total[PER], sum = 0;
#pragma unroll
  for (int q = 0; q < PER; ++q) before[q] = total[q] = 0;
  if (tid * PER < R) {
    if (ntiles <= RS_DIRECT) {
      // eight tiles' counts in flight at a time
      for (int t0 = 0; t0 < ntiles; t0 += 8) {
        int h[8][PER];
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
          for (int q = 0; q < PER; ++q)
            h[t][q] = t0 + t < ntiles && tid * PER + q < R ? hist[(size_t)(t0 + t) * R + tid * PER + q] : 0;
#pragma unroll
        for (int t = 0; t < 8; ++t)
#pragma unroll
          for (int q = 0; q < PER; ++q) {
            total[q] += h[t][q];
            before[q] += t0 + t < tile ? h[t][q] : 0;
          }
      }
    } else {
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int d = tid * PER + q;
        if (d < R) {
          before[q] = hist[(size_t)tile * R + d];
          total[q] = tot[d];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) sum += total[q];
  }
  int all;
  int run = block_exclusive(sum, &all);  // (its barriers also end the clearing)
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (tid * PER + q < R) base[tid * PER + q] = run + before[q];
    run += total[q];
  }
  __syncthreads();
  const uint64_t lt = (1ull << lane) - 1;
  int rk[RS_ITEMS];
#pragma unroll
  for (int j = 0; j < RS_ITEMS; ++j) {
    const bool valid = i0 + j * 64 < n;
    const uint32_t d = digit_of(kk[j], shift, width);
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < RS_MAX_DIGIT; ++b) {
      const uint64_t bal = __ballot((d >> b) & 1u);
      m &= ((d >> b) & 1u) ? bal : ~bal;
    }
    const int prev = wcnt[wid][d], rank = __popcll(m & lt);
    if (valid && rank == 0) wcnt[wid][d] = (uint16_t)(prev + __popcll(m));
    rk[j] = prev + rank;
  }
  __syncthreads();
  // counts to places among the waves
  for (int d = tid; d < R; d += RS_BLOCK) {
    int r = 0;
#pragma unroll
    for (int w = 0; w < RS_WAVES; ++w) {
      const int c = wcnt[w][d];
      wcnt[w][d] = (uint16_t)r;
      r += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < RS_ITEMS; ++j) {
    if (i0 + j * 64 >= n) continue;
    const uint32_t d = digit_of(kk[j], shift, width);
    const int off = base[d] + wcnt[wid][d] + rk[j];
    kout[off] = kk[j];
    vout[off] = vv[j];
  }
}

int sort_hist_size(int cap, int digit_bits) {
  return (1 << digit_bits) * ((int)(((long long)cap + RS_TILE - 1) / RS_TILE) + 1);
}

template <typename Key>
Sorted<Key> radix_sort(Key *k0, uint32_t *v0, Key *k1, uint32_t *v1, int cap, const int32_t *d_n, int bits,
                       int digit_bits, int32_t *hist, hipStream_t s) {
  Key *ka = k0, *kb = k1;
  uint32_t *va = v0, *vb = v1;
  if (cap <= 0) return {ka, va};
  const int ntiles = (int)(((long long)cap + RS_TILE - 1) / RS_TILE);
  const int passes = (bits + digit_bits - 1) / digit_bits, width = (bits + passes - 1) / passes;
  int32_t *tot = hist + ((size_t)ntiles << width);
  for (int q = 0; q < passes; ++q) {
    const int shift = q * width;
    hipLaunchKernelGGL(k_rs_hist<Key>, dim3(ntiles), dim3(RS_BLOCK), 0, s, ka, cap, d_n, shift, width, hist);
    if (ntiles > RS_DIRECT)
      hipLaunchKernelGGL(k_rs_cols, dim3(((1 << width) + 63) / 64), dim3(1024), 0, s, cap, d_n, width, hist, tot);
    hipLaunchKernelGGL(k_rs_scatter<Key>, dim3(ntiles), dim3(RS_BLOCK), 0, s, ka, va, cap, d_n, shift, width, hist,
                       tot, kb, vb);
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  return {ka, va};
}
template Sorted<uint64_t> radix_sort<uint64_t>(uint64_t *, uint32_t *, uint64_t *, uint32_t *, int, const int32_t *,
                                               int, int, int32_t *, hipStream_t);
template Sorted<uint32_t> radix_sort<uint32_t>(uint32_t *, uint32_t *, uint32_t *, uint32_t *, int, const int32_t *,
                                               int, int, int32_t *, hipStream_t);

// ------------------------------------------------------ packed positions
__global__ void k_pack_xy(const float *__restrict__ x, const float *__restrict__ y, float2 *__restrict__ xy, int n,
                          int32_t *__restrict__ bad, int32_t gen, const int32_t *__restrict__ err,
                          uint32_t *__restrict__ tag, uint32_t *__restrict__ note, uint32_t noted) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (note && i == 0) *note = noted;
  if (tag && i == 0) {
    // whether a sweep gave up (bit 1) since the last arrival pass began: the word is cleared after this
    const uint32_t gave_up = tag[3] | (*err & 2) >> 1;
    if (note) {  // a new arrival pass
      tag[0] = tag[0] + 1;
      tag[1] = gave_up;
    }
    tag[3] = note ? 0 : gave_up;
  }
  if (i >= n) return;
  const float a = x[i], b = y[i];
  xy[i] = make_float2(a, b);
  // every writer stores the same value, so no atomic is needed
  if (bad && !(__builtin_isfinite(a) && __builtin_isfinite(b))) *bad = gen;
}
void pack_xy(const float *x, const float *y, float2 *xy, int n, hipStream_t s, int32_t *bad, int32_t gen,
             const int32_t *err, uint32_t *tag, uint32_t *note, uint32_t noted) {
  if (n > 0)
    hipLaunchKernelGGL(k_pack_xy, dim3((n + 255) / 256), dim3(256), 0, s, x, y, xy, n, bad, gen, err, tag, note,
                       noted);
}

// ---------------------------------------------------------- small fills
__global__ void k_fill_i32(int32_t *p, int n, int32_t v) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
void fill_i32(int32_t *p, int n, int32_t v, hipStream_t s) {
  if (n > 0) hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, s, p, n, v);
}

}  // namespace tdp
