// Per-box precomputation, summed-area tables in HBM, the box kernels that read
// those tables, and the box-gradient reduction.  gfx950, wave64.
#include "bc_box.hpp"

#include <algorithm>

namespace bc {

// ---------------------------------------------------------------------------
// Kernels
// ---------------------------------------------------------------------------
// Tap records (16 words each): record r < CB is box r's forward taps, record
// CB + r its adjoint taps (make_taps_adjoint); with `rounded`, the taps of
// the boxes with rounded (integer) corners and of their adjoints.
__global__ void k_box_prep(const float* __restrict__ boxes, int CB, int rounded, int* __restrict__ table) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 2 * CB) return;
  const bool adj = i >= CB;
  const float* p = boxes + (size_t)(adj ? i - CB : i) * 4;
  const Taps<float> t = rounded ? make_taps_rounded(p, adj, 1 << 20, 1 << 20)
                        : adj   ? make_taps_adjoint(p, 1 << 20, 1 << 20)
                                : make_taps_f32(p, false, 1 << 20, 1 << 20);
  int* r = table + (size_t)i * 16;
  float* f = reinterpret_cast<float*>(r);
  r[0] = t.ox[0]; r[1] = t.ox[2]; r[2] = t.oy[0]; r[3] = t.oy[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) { f[4 + k] = t.wx[k]; f[8 + k] = t.wy[k]; r[12 + k] = 0; }
}

// Box-parameter reparameterisation (Section 3.2): corners kept as u in
// [-1, 1] relative to a maximum box size M per axis, x_l = u_xl * M_x / 2,
// x_h = u_xh * M_x / 2, box [x + x_l, x + x_h + 1).  fp64 arithmetic (exact
// for these operands), rounded once to fp32.
__global__ void k_boxes_from_unit(const float* __restrict__ u, int n, float mw, float mh,
                                  float* __restrict__ boxes) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* q = u + (size_t)i * 4;
  const double xl = (double)q[0] * (double)mw / 2, xh = (double)q[1] * (double)mw / 2;
  const double yl = (double)q[2] * (double)mh / 2, yh = (double)q[3] * (double)mh / 2;
  *reinterpret_cast<float4*>(boxes + (size_t)i * 4) =
      make_float4((float)((xl + xh) / 2), (float)((yl + yh) / 2), (float)((xh - xl + 1) / 2), (float)((yh - yl + 1) / 2));
}

// dL/du from dL/d(cx, cy, rx, ry) through the map above: x_l = a and
// x_h = b - 1 with cx = (a + b - 1) / 2, rx = (b - a) / 2.
__global__ void k_unit_grad(const float* __restrict__ g, int n, float mw, float mh, float* __restrict__ gu) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float4 q = *reinterpret_cast<const float4*>(g + (size_t)i * 4);
  const double sx = (double)mw / 2, sy = (double)mh / 2;
  *reinterpret_cast<float4*>(gu + (size_t)i * 4) =
      make_float4((float)(((double)q.x - q.z) / 2 * sx), (float)(((double)q.x + q.z) / 2 * sx),
                  (float)(((double)q.y - q.w) / 2 * sy), (float)(((double)q.y + q.w) / 2 * sy));
}

// After an update: clip u to [-1, 1] and swap a reversed corner pair.
__global__ void k_clip_unit(float* __restrict__ u, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float4 q = *reinterpret_cast<float4*>(u + (size_t)i * 4);
  q.x = fminf(fmaxf(q.x, -1.f), 1.f); q.y = fminf(fmaxf(q.y, -1.f), 1.f);
  q.z = fminf(fmaxf(q.z, -1.f), 1.f); q.w = fminf(fmaxf(q.w, -1.f), 1.f);
  *reinterpret_cast<float4*>(u + (size_t)i * 4) = make_float4(fminf(q.x, q.y), fmaxf(q.x, q.y), fminf(q.z, q.w),
                                                              fmaxf(q.z, q.w));
}

// Standalone table in HBM, one block per map.  The map is processed in strips
// of kStrip rows staged in LDS: each wave scans whole rows (every lane holds a
// run of consecutive elements, scanned serially, then a wave-level scan of
// the lane totals), then lanes own columns and carry the column sums down the
// strip, writing finished table rows coalesced.
constexpr int kStrip = 16;
constexpr int kSatMaxK = 16;  // elements per lane in a row scan: W <= 1024
constexpr int kSatRowsPerWave = 4;  // rows of a strip each wave loads before scanning them

// kUp: x is [maps][Ho][Wo] and the table is that of its zero-upsampled H x W
// map (x[i][j] at (s*i, s*j)); mean must then be null.
// KM: elements per lane in a row scan, K = ceil(W / 64) <= KM (4 for
// W <= 256, 8 for W <= 512, else 16).  kGroups > 1 (W <= 256, few maps): blocks of
// 256 * kGroups threads take strips of kStrip * kGroups rows, and the column
// pass runs kGroups row groups of kStrip rows in parallel, each starting from
// the carried sums plus the totals of the groups above it.
// kBands (few maps): a map's rows are divided over gridDim.x / maps blocks of
// band_rows rows each; bands holds the column sums of every band
// (k_sat_bands), from which a block forms the table row above its band, and
// mean is read, not computed.
template <typename T, bool kUp, int KM, int kGroups, bool kBands = false>
__global__ __launch_bounds__(256 * kGroups) void k_sat_build(const T* __restrict__ x, T* __restrict__ sat,
                                                             float* __restrict__ mean, int H, int W, int s, int Ho,
                                                             int Wo, const T* __restrict__ bands = nullptr,
                                                             int nbands = 1, int band_rows = 0, int total = 0) {
  static_assert(kGroups == 1 || KM == 4, "row groups need W <= 256");
  constexpr int kRowsStrip = kStrip * kGroups;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* tile = reinterpret_cast<T*>(smem_raw);
  __shared__ float red[16];
  __shared__ T part[kGroups > 1 ? kGroups * 256 : 1];
  int map = blockIdx.x, band = 0;
  if constexpr (kBands) {
    const int L = xcd_remap(blockIdx.x, gridDim.x);
    if (L >= total) return;
    map = L / nbands;
    band = L - map * nbands;
  }
  const T* src = x + (size_t)map * (kUp ? (size_t)Ho * Wo : (size_t)H * W);
  T* dst = sat + (size_t)map * (H + 1) * (W + 1);
  float mu = 0.f;
  const bool sub = mean != nullptr;
  if (sub && kBands) {
    mu = mean[map];
  } else if (sub) {
    mu = block_mean(reinterpret_cast<const float*>(src), H * W, red);
    if (threadIdx.x == 0) mean[map] = mu;
  }
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int K = (W + 63) >> 6;
  if (band == 0)
    for (int v = tid; v <= W; v += blockDim.x) dst[v] = (T)0;
  T carry[KM / 4];
#pragma unroll
  for (int j = 0; j < KM / 4; ++j) carry[j] = (T)0;
  const int r_begin = kBands ? band * band_rows : 0, r_end = kBands ? min(H, r_begin + band_rows) : H;
  if (kBands && band > 0) {
    // the table row above this band: the column sums of the bands above,
    // scanned like a row of the map
    for (int v = tid; v < W; v += blockDim.x) {
      T above = (T)0;
      if (!kUp || v % s == 0) {
        const T* col = bands + (size_t)map * nbands * (kUp ? Wo : W) + (kUp ? v / s : v);
#pragma unroll 4
        for (int h = 0; h < band; ++h) above += col[(size_t)h * (kUp ? Wo : W)];
      }
      tile[v] = above;
    }
    __syncthreads();
    if (wave == 0) {
      T v[KM], run = (T)0;
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        const int idx = lane * K + k;
        if (k < K) {
          run += idx < W ? tile[idx] : (T)0;
          v[k] = run;
        }
      }
      const T excl = group_excl<64>(run);
#pragma unroll
      for (int k = 0; k < KM; ++k) {
        const int idx = lane * K + k;
        if (k < K && idx < W) tile[idx] = v[k] + excl;
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < KM / 4; ++j) {
      const int v = (kGroups == 1 ? tid : tid & 255) + j * 256;
      if (v < W) carry[j] = tile[v];
    }
    __syncthreads();
  }
  for (int r0 = r_begin; r0 < r_end; r0 += kRowsStrip) {
    const int rows = min(kRowsStrip, r_end - r0);
    // rows rr = wave + i * nw of the strip: all of a wave's loads are issued
    // before its first scan
    for (int rb = wave; rb < rows; rb += kSatRowsPerWave * nw) {
      T v[kSatRowsPerWave][KM];
#pragma unroll
      for (int i = 0; i < kSatRowsPerWave; ++i) {
        const int rr = rb + i * nw, r = r0 + rr;
        const T* row = kUp ? src + (size_t)(r / s) * Wo : src + (size_t)r * W;
        const bool live = rr < rows && (!kUp || r % s == 0);
#pragma unroll
        for (int k = 0; k < KM; ++k) {
          if (k < K) {
            const int idx = lane * K + k;
            T val;
            if constexpr (kUp) val = (live && idx < W && idx % s == 0) ? row[idx / s] : (T)0;
            else val = (live && idx < W) ? row[idx] : (T)0;
            if (sub && idx < W) val = (T)((float)val - mu);
            v[i][k] = val;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < kSatRowsPerWave; ++i) {
        const int rr = rb + i * nw;
        T run = (T)0;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
          if (k < K) {
            run += v[i][k];
            v[i][k] = run;
          }
        }
        const T excl = group_excl<64>(run);
        if (rr < rows) {
#pragma unroll
          for (int k = 0; k < KM; ++k) {
            const int idx = lane * K + k;
            if (k < K && idx < W) tile[rr * W + idx] = v[i][k] + excl;
          }
        }
      }
    }
    __syncthreads();
    if constexpr (kGroups == 1) {
#pragma unroll
      for (int j = 0; j < KM / 4; ++j) {
        const int v = tid + j * 256;
        if (v < W) {
          T cs = carry[j];
          for (int rr = 0; rr < rows; ++rr) {
            cs += tile[rr * W + v];
            dst[(size_t)(r0 + rr + 1) * (W + 1) + v + 1] = cs;
          }
          carry[j] = cs;
        }
      }
    } else {
      // column v, row group g: rows [g * kStrip, (g + 1) * kStrip) of the strip
      const int v = tid & 255, g = tid >> 8;
      const int ra = g * kStrip, rz = min(ra + kStrip, rows);
      T ps = (T)0;
      if (v < W)
        for (int rr = ra; rr < rz; ++rr) ps += tile[rr * W + v];
      part[g * 256 + v] = ps;
      __syncthreads();
      if (v < W) {
        T cs = carry[0], tot = (T)0;
#pragma unroll
        for (int h = 0; h < kGroups; ++h) {
          const T p = part[h * 256 + v];
          if (h < g) cs += p;
          tot += p;
        }
        for (int rr = ra; rr < rz; ++rr) {
          cs += tile[rr * W + v];
          dst[(size_t)(r0 + rr + 1) * (W + 1) + v + 1] = cs;
        }
        carry[0] += tot;
      }
    }
    if (tid < rows) dst[(size_t)(r0 + tid + 1) * (W + 1)] = (T)0;
    __syncthreads();
  }
}

// Column sums of each band of band_rows rows of each map (minus the map's
// mean, if given): bands[map][band][column of x].  One block per (map, band).
template <typename T, bool kUp>
__global__ __launch_bounds__(256) void k_sat_bands(const T* __restrict__ x, T* __restrict__ bands,
                                                   const float* __restrict__ mean, int H, int W, int s, int Ho, int Wo,
                                                   int nbands, int band_rows, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int map = L / nbands, band = L - map * nbands;
  const int r0 = band * band_rows, r1 = min(H, r0 + band_rows);
  const int i0 = kUp ? (r0 + s - 1) / s : r0, i1 = kUp ? (r1 + s - 1) / s : r1, cols = kUp ? Wo : W;
  const T* src = x + (size_t)map * (kUp ? (size_t)Ho * Wo : (size_t)H * W);
  const float mu = mean != nullptr ? mean[map] : 0.f;
  for (int v = threadIdx.x; v < cols; v += 256) {
    T sum = (T)0;
#pragma unroll 8
    for (int i = i0; i < i1; ++i) {
      const T t = src[(size_t)i * cols + v];
      sum += mean != nullptr ? (T)((float)t - mu) : t;
    }
    bands[(size_t)L * cols + v] = sum;
  }
}

// Mean of each map.
__global__ __launch_bounds__(1024) void k_map_mean(const float* __restrict__ x, float* __restrict__ mean, int n) {
  __shared__ float red[16];
  const float mu = block_mean(x + (size_t)blockIdx.x * n, n, red);
  if (threadIdx.x == 0) mean[blockIdx.x] = mu;
}

// Forward, table in HBM: one block per (map, box, block of 256 items), mapped
// so that one map's blocks run on one XCD.
template <typename T, typename OutT, int SEG, bool kOffset, bool kInt, bool kNT>
__global__ __launch_bounds__(256) void k_box_fwd_gather(const T* __restrict__ sat, const float* __restrict__ means,
                                                        const int* __restrict__ taps, OutT* __restrict__ y,
                                                        int C, int H, int W, int B, int nblk, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int blk = L % nblk, mb = L / nblk;
  const int b = mb % B, map = mb / B, c = map % C;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const int it = blk * 256 + threadIdx.x;
  if (it >= nch * nseg) return;
  const int seg = it / nch, ch = it - seg * nch;
  const GlobalTable<T, true> tab{sat + (size_t)map * (H + 1) * (W + 1), W + 1, W, H};
  const float mu = kOffset ? means[map] : 0.f;
  const Taps<T> tp = typed_taps<T>(load_taps(taps + (size_t)(c * B + b) * 16, W, H));
  OutT* out = y + ((size_t)map * B + b) * H * W;
  const int x0 = ch * kQ, y0 = seg * SEG, y1 = min(y0 + SEG, H);
  StoreRows<OutT, T, kNT> em{out, W, x0, y0 * W + x0};
  if (y0 + SEG <= H && x0 + kQ <= W) walk_fwd<SEG, T, kOffset, true, kInt>(tab, tp, H, W, x0, y0, y1, mu, em);
  else walk_fwd<SEG, T, kOffset, false, kInt>(tab, tp, H, W, x0, y0, y1, mu, em);
}

// Strided forward, table in HBM: one block per (map, box, block of 256 items).
template <typename T, typename OutT, bool kOffset, bool kInt>
__global__ __launch_bounds__(256) void k_box_fwd_gather_strided(const T* __restrict__ sat,
                                                                const float* __restrict__ means,
                                                                const int* __restrict__ taps, OutT* __restrict__ y,
                                                                int C, int H, int W, int B, int s, int Ho, int Wo,
                                                                int nblk, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int blk = L % nblk, mb = L / nblk;
  const int b = mb % B, map = mb / B, c = map % C;
  const int it = blk * 256 + threadIdx.x;
  if (it >= Wo * ((Ho + kSegS - 1) / kSegS)) return;
  const int seg = it / Wo, j = it - seg * Wo;
  const GlobalTable<T, true> tab{sat + (size_t)map * (H + 1) * (W + 1), W + 1, W, H};
  const float mu = kOffset ? means[map] : 0.f;
  const Taps<T> tp = typed_taps<T>(load_taps(taps + (size_t)(c * B + b) * 16, W, H));
  const int i0 = seg * kSegS;
  StoreCol<OutT, T> em{y + ((size_t)map * B + b) * Ho * Wo, Wo, i0 * Wo + j};
  box_walk_strided<kSegS, T, kOffset, kInt>(tab, tp, H, W, s * j, i0, min(i0 + kSegS, Ho), s, mu, em);
}

// Backward, tables in HBM (one table per gradient map, built beforehand).
// One 256-thread block per (map, block of 256 items); loops over boxes.
// partials: [((n * nblk + blk) * 4 + wave) * C*B + c*B + b][4]; kInt as in
// k_box_bwd_lds.  Four waves per SIMD: without the ReLU that takes exactly the 128
// VGPRs allowed, with it 129, so there the bound is set (3 x 63 maps of 106x583,
// 4 boxes: 414 us without, 400 with).
template <int SEG, bool kInt, bool kRelu>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kRelu ? 4 : 3, 8))) void k_box_bwd_gather(
    const float* __restrict__ x, const float* __restrict__ sat_g, const int* __restrict__ taps, void* __restrict__ gx,
    float* __restrict__ partials, int C, int H, int W, int B, int nblk, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int blk = L % nblk, map = L / nblk;
  const int n = map / C, c = map - n * C;
  const int wave = threadIdx.x >> 6;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const int it = blk * 256 + threadIdx.x;
  const bool active = it < nch * nseg;
  const int seg = it / nch, ch = it - seg * nch;
  const int x0 = ch * kQ, y0 = seg * SEG, y1 = min(y0 + SEG, H);
  const bool full = y0 + SEG <= H && x0 + kQ <= W;
  const size_t tsz = (size_t)(H + 1) * (W + 1);
  float v[SEG][kQ], acc[SEG][kQ];
  if constexpr (!kInt) load_item<SEG>(x + (size_t)map * H * W, H, W, x0, y0, active, v);
  uint32_t rmask = 0;
  if constexpr (kRelu) rmask = relu_mask<SEG>(v);
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[s][q] = 0.f;
  const int* adj = taps + (size_t)C * B * 16;
  for (int b = 0; b < B; ++b) {
    const GlobalTable<float> tg{sat_g + ((size_t)map * B + b) * tsz, W + 1, W, H};
    const Taps<float> tp = load_taps(adj + (size_t)(c * B + b) * 16, W, H);
    if constexpr (kInt) {  // integer corners: input gradient only
      AccRows<SEG> em{acc};
      if (active) {
        if (full) box_walk_int<SEG, float, false, true>(tg, tp, H, W, x0, y0, y1, 0.f, em);
        else box_walk_int<SEG, float, false, false>(tg, tp, H, W, x0, y0, y1, 0.f, em);
      }
      continue;
    }
    float E[4] = {0.f, 0.f, 0.f, 0.f};
    if (active) {
      if (full) adjoint_walk<SEG, true>(tg, tp, x0, y0, y1, v, acc, E);
      else adjoint_walk<SEG, false>(tg, tp, x0, y0, y1, v, acc, E);
    }
    float g4[4] = {-E[1], E[0], -E[3], E[2]};   // dL/da, dL/db, dL/dc, dL/dd
    store_wave_partial(g4, partials + ((((size_t)n * nblk + blk) * 4 + wave) * C * B + (size_t)c * B + b) * 4);
  }
  if (active && gx != nullptr) {
    if constexpr (kRelu) store_item_relu_bf16<SEG>(static_cast<uint16_t*>(gx) + (size_t)map * H * W, H, W, x0, y0, acc, rmask);
    else store_item<SEG>(static_cast<float*>(gx) + (size_t)map * H * W, H, W, x0, y0, acc);
  }
}

// Second stage of the box-parameter gradient: fixed-order sum of the partial
// edge gradients, then the change of variables a = 1/2+cx-rx, b = 1/2+cx+rx,
// c = 1/2+cy-ry, d = 1/2+cy+ry:  dcx = ga+gb, dcy = gc+gd, drx = gb-ga,
// dry = gd-gc.
// One block per 16 boxes: thread (q, j) sums rows p = q, q + 16, ... of box
// j (a wave's load covers 4 rows x 16 consecutive boxes, 256 contiguous
// bytes each), then the 16 row-sums of each box combine in a fixed tree
// (lane shuffles across the wave's 4 row groups, then the 4 waves in LDS).
__global__ __launch_bounds__(256) void k_box_grad_reduce(const float* __restrict__ partials, int P, int CB,
                                                         float* __restrict__ out) {
  __shared__ float4 red[4][kReduceBoxes];
  const int j = threadIdx.x % kReduceBoxes, q = threadIdx.x / kReduceBoxes;
  const int i = blockIdx.x * kReduceBoxes + j;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < CB)
    for (int p = q; p < P; p += 256 / kReduceBoxes) {
      const float4 v = *reinterpret_cast<const float4*>(partials + ((size_t)p * CB + i) * 4);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
#pragma unroll
  for (int m = 16; m < 64; m <<= 1) {
    s.x += __shfl_xor(s.x, m); s.y += __shfl_xor(s.y, m);
    s.z += __shfl_xor(s.z, m); s.w += __shfl_xor(s.w, m);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) < kReduceBoxes) red[wave][j] = s;
  __syncthreads();
  if (threadIdx.x < kReduceBoxes && i < CB) {
    float4 t = red[0][j];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      const float4 u = red[w][j];
      t.x += u.x; t.y += u.y; t.z += u.z; t.w += u.w;
    }
    *reinterpret_cast<float4*>(out + (size_t)i * 4) = make_float4(t.x + t.y, t.z + t.w, t.y - t.x, t.w - t.z);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_box_prep(const float* boxes, int C, int B, bool rounded, void* table, hipStream_t s) {
  const int n = 2 * C * B;
  hipLaunchKernelGGL(k_box_prep, dim3((n + 255) / 256), dim3(256), 0, s, boxes, C * B, (int)rounded, (int*)table);
  return last_error();
}

hipError_t launch_unit_params(int op, const float* in, int n, float mw, float mh, float* out, hipStream_t s) {
  const dim3 grid((n + 255) / 256), block(256);
  if (op == 0) hipLaunchKernelGGL(k_boxes_from_unit, grid, block, 0, s, in, n, mw, mh, out);
  else if (op == 1) hipLaunchKernelGGL(k_unit_grad, grid, block, 0, s, in, n, mw, mh, out);
  else hipLaunchKernelGGL(k_clip_unit, grid, block, 0, s, out, n);
  return last_error();
}

// Maps too few to fill the chip with one block each: up to 256 wide they take
// blocks of 1024 threads over 64-row strips; wider ones, with scratch for the
// column sums of each band, are divided over enough blocks for 8 per CU (one
// block walks the strips of its map one after another, 9 us each: 2 x 32 maps of
// 288x384 157 us, divided 24 us).  Dividing reads the map twice, which costs more
// than it fills from little more than a block per CU on, or, where the mean is
// read first and so costs as much anyway, from about three (us of a call with
// whole and with divided tables; backward, 1 box: 256 maps of 162x680 273, 256;
// 400 384, 431; 600 567, 660; 256 of 288x384 257, 214; 400 359, 367; 600 488, 569;
// forward with the mean, 4 boxes: 400 of 288x384 660, 499; 700 963, 963).
constexpr int kSatBandMaps = 320, kSatBandMapsMean = 640, kSatBandBlocks = 2048;
constexpr int kSatFewMaps = 2048;

template <typename T, bool kUp>
static void sat_build_t(const T* x, T* sat, float* mean, int maps, int H, int W, int stride, SatScratch scratch,
                        hipStream_t s) {
  const int Ho = (H + stride - 1) / stride, Wo = (W + stride - 1) / stride, cols = kUp ? Wo : W;
  const bool divide = W > 256 && maps < (mean ? kSatBandMapsMean : kSatBandMaps);
  int nb = divide ? std::min((kSatBandBlocks + maps - 1) / maps, (H + kStrip - 1) / kStrip) : 1;
  nb = (int)std::min<size_t>(nb, scratch.bytes / ((size_t)maps * cols * 4));
  if (nb > 1) {
    const int band_rows = ((H + nb * kStrip - 1) / (nb * kStrip)) * kStrip;
    nb = (H + band_rows - 1) / band_rows;
    const int total = maps * nb;
    T* bands = static_cast<T*>(scratch.p);
    if (mean)
      hipLaunchKernelGGL(k_map_mean, dim3(maps), dim3(1024), 0, s, reinterpret_cast<const float*>(x), mean, H * W);
    hipLaunchKernelGGL((k_sat_bands<T, kUp>), dim3(pad8(total)), dim3(256), 0, s, x, bands, mean, H, W, stride, Ho, Wo,
                       nb, band_rows, total);
    auto go = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(pad8(total)), dim3(256), (size_t)kStrip * W * 4, s, x, sat, mean, H, W, stride, Ho,
                         Wo, (const T*)bands, nb, band_rows, total);
    };
    if (W <= 512) go(k_sat_build<T, kUp, 8, 1, true>);
    else go(k_sat_build<T, kUp, kSatMaxK, 1, true>);
    return;
  }
  auto go = [&](auto kernel, int groups) {
    hipLaunchKernelGGL(kernel, dim3(maps), dim3(256 * groups), (size_t)kStrip * groups * W * 4, s, x, sat, mean, H, W,
                       stride, Ho, Wo, (const T*)nullptr, 1, 0, 0);
  };
  if (W > 512) go(k_sat_build<T, kUp, kSatMaxK, 1>, 1);
  else if (W > 256) go(k_sat_build<T, kUp, 8, 1>, 1);
  else if (maps < kSatFewMaps && !kUp) go(k_sat_build<T, kUp, 4, kUp ? 1 : 4>, 4);
  else go(k_sat_build<T, kUp, 4, 1>, 1);
}

hipError_t launch_sat_build(const void* x, bool is_int, void* sat, float* mean, int maps, int H, int W,
                            SatScratch scratch, hipStream_t s) {
  if (is_int) sat_build_t<int, false>((const int*)x, (int*)sat, nullptr, maps, H, W, 1, scratch, s);
  else sat_build_t<float, false>((const float*)x, (float*)sat, mean, maps, H, W, 1, scratch, s);
  return last_error();
}

hipError_t launch_sat_build_up(const float* x, float* sat, int maps, int H, int W, int stride, SatScratch scratch,
                               hipStream_t s) {
  sat_build_t<float, true>(x, sat, nullptr, maps, H, W, stride, scratch, s);
  return last_error();
}

template <typename T, typename OutT, bool kOffset>
static void fwd_gather_t(const void* sat, const float* means, const int* taps, void* y, int N, int C, int H, int W,
                         int B, bool rounded, int stride, hipStream_t s) {
  constexpr int SEG = 16;
  if (stride == 1) {
    const int items = n_chunks(W) * n_segs(H, SEG);
    const int nblk = (items + 255) / 256;
    const int total = N * C * B * nblk;
    const bool nt = stream_out((size_t)N * C * B * H * W, sizeof(OutT));
    with_flag(rounded, [&](auto ki) {
      with_flag(nt, [&](auto kn) {
        hipLaunchKernelGGL((k_box_fwd_gather<T, OutT, SEG, kOffset, decltype(ki)::value, decltype(kn)::value>),
                           dim3(pad8(total)), dim3(256), 0, s, (const T*)sat, means, taps, (OutT*)y, C, H, W, B, nblk,
                           total);
      });
    });
    return;
  }
  const int Ho = (H + stride - 1) / stride, Wo = (W + stride - 1) / stride;
  const int nblk = (Wo * ((Ho + kSegS - 1) / kSegS) + 255) / 256;
  const int total = N * C * B * nblk;
  with_flag(rounded, [&](auto ki) {
    hipLaunchKernelGGL((k_box_fwd_gather_strided<T, OutT, kOffset, decltype(ki)::value>), dim3(pad8(total)),
                       dim3(256), 0, s, (const T*)sat, means, taps, (OutT*)y, C, H, W, B, stride, Ho, Wo, nblk,
                       total);
  });
}

hipError_t launch_box_fwd_gather(const void* sat, bool is_int, const float* means, const int* taps, void* y,
                                 int out_kind, int N, int C, int H, int W, int B, bool rounded, int stride,
                                 hipStream_t s) {
  const bool offset = means != nullptr;
  if (is_int) {
    fwd_gather_t<int, int, false>(sat, nullptr, taps, y, N, C, H, W, B, rounded, stride, s);
  } else if (out_kind == 2) {
    if (offset) fwd_gather_t<float, uint16_t, true>(sat, means, taps, y, N, C, H, W, B, rounded, stride, s);
    else fwd_gather_t<float, uint16_t, false>(sat, nullptr, taps, y, N, C, H, W, B, rounded, stride, s);
  } else {
    if (offset) fwd_gather_t<float, float, true>(sat, means, taps, y, N, C, H, W, B, rounded, stride, s);
    else fwd_gather_t<float, float, false>(sat, nullptr, taps, y, N, C, H, W, B, rounded, stride, s);
  }
  return last_error();
}

int box_bwd_gather_blocks(int H, int W) { return (n_chunks(W) * n_segs(H, kBwdGatherSeg) + 255) / 256; }

hipError_t launch_box_bwd_gather(const float* x, const float* sat_g, const int* taps, void* gx, float* partials,
                                 int N, int C, int H, int W, int B, bool rounded, bool relu_bf16, hipStream_t s) {
  if (rounded && relu_bf16) return hipErrorInvalidValue;
  const int nblk = box_bwd_gather_blocks(H, W);
  const int total = N * C * nblk;
  auto go = [&](auto ki, auto kr) {
    hipLaunchKernelGGL((k_box_bwd_gather<kBwdGatherSeg, decltype(ki)::value, decltype(kr)::value>), dim3(pad8(total)),
                       dim3(256), 0, s, x, sat_g, taps, gx, partials, C, H, W, B, nblk, total);
  };
  if (rounded) go(std::true_type{}, std::false_type{});
  else with_flag(relu_bf16, [&](auto kr) { go(std::false_type{}, kr); });
  return last_error();
}

hipError_t launch_box_grad_reduce(const float* partials, int P, int CB, float* grad_boxes, hipStream_t s) {
  hipLaunchKernelGGL(k_box_grad_reduce, dim3((CB + kReduceBoxes - 1) / kReduceBoxes), dim3(256), 0, s, partials, P, CB,
                     grad_boxes);
  return last_error();
}

}  // namespace bc
