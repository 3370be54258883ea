// Kernel splitting: box filter kernels of boxes cut into weighted pieces,
// tables in LDS or HBM.  gfx950, wave64.
#include "bc_box.hpp"

namespace bc {
// ---------------------------------------------------------------------------
// Kernel splitting (Section 3.1, Fig. 2): a box cut at its centre line(s)
// m = (a + b) / 2, n = (c + d) / 2 into nx * ny pieces with their own
// weights; the output is the weighted sum of the pieces' box sums.
// ---------------------------------------------------------------------------
// Corner records of split boxes for the forward, 32 words per box: a split
// box is sum_{i,j} w_ij * (box sum over [k_j, k_{j+1}) x [r_i, r_{i+1})), and
// each piece's box sum is the four-corner difference of the interpolated
// table, so the whole box is sum over the (nx+1) x (ny+1) shared corners of
// coef(ri, kj) * T(r_ri, k_kj) with
//   coef(ri, kj) = w(ri-1, kj-1) - w(ri-1, kj) - w(ri, kj-1) + w(ri, kj)
// (w = 0 outside the pieces): 9 interpolated corners for 4 pieces instead of
// 16.  Words: 0..2 column-corner floors, 3..5 row-corner floors, 6..11 row
// weights (1 - beta, beta) per row corner, 12..29 column weights
// coef * (1 - alpha), coef * alpha per (row corner, column corner); fp64
// edges and products, each weight rounded once.
__global__ void k_box_prep_corners(const float* __restrict__ boxes, const float* __restrict__ piece_w, int CB,
                                   int nx, int ny, int* __restrict__ table) {
  const int box = blockIdx.x * blockDim.x + threadIdx.x;
  if (box >= CB) return;
  const float* q = boxes + (size_t)box * 4;
  const double cx = q[0], cy = q[1], rx = q[2], ry = q[3];
  const double a = 0.5 + cx - rx, b = 0.5 + cx + rx, c = 0.5 + cy - ry, d = 0.5 + cy + ry;
  const double ke[3] = {a, nx == 2 ? (a + b) / 2 : b, b};
  const double re[3] = {c, ny == 2 ? (c + d) / 2 : d, d};
  const float* wp = piece_w + (size_t)box * nx * ny;
  auto w = [&](int i, int j) -> double {
    return (i < 0 || j < 0 || i >= ny || j >= nx) ? 0.0 : (double)wp[i * nx + j];
  };
  int* r = table + (size_t)box * 32;
  float* f = reinterpret_cast<float*>(r);
  double alpha[3];
  for (int k = 0; k <= nx; ++k) {
    int fl;
    edge_split(ke[k], 1 << 20, fl, alpha[k]);
    r[k] = fl;
  }
  for (int i = 0; i <= ny; ++i) {
    int fl;
    double beta;
    edge_split(re[i], 1 << 20, fl, beta);
    r[3 + i] = fl;
    f[6 + 2 * i] = (float)(1.0 - beta);
    f[7 + 2 * i] = (float)beta;
    for (int k = 0; k <= nx; ++k) {
      const double cf = w(i - 1, k - 1) - w(i - 1, k) - w(i, k - 1) + w(i, k);
      f[12 + (i * 3 + k) * 2] = (float)(cf * (1.0 - alpha[k]));
      f[13 + (i * 3 + k) * 2] = (float)(cf * alpha[k]);
    }
  }
  for (int k = 30; k < 32; ++k) r[k] = 0;
}

// Forward walk of a split box over its shared corners (record above), on a
// map's table in LDS: per table row v and row corner ri the column-weighted
// row R_ri(v)[q] = sum_kj cw0 * S(v, x+f_kj) + cw1 * S(v, x+f_kj+1), and the
// output of row y is sum_ri (1-beta) R_ri(y+f_ri) + beta R_ri(y+f_ri+1).
// Each step reads one new table row per row corner (NXC runs of kQ+1 words)
// and reuses the one from the step before.
template <int SEG, int NXC, int NYC, bool kFull, typename Src, typename Emit>
__device__ __forceinline__ void corner_walk(const Src& S, const int* __restrict__ rec, int x0, int y0, int y1,
                                            Emit& emit) {
  const float* f = reinterpret_cast<const float*>(rec);
  const int W = S.W, H = S.H;
  typename Src::Col col[NXC];
  float cw[NYC][NXC][2], wy[NYC][2];
  int rc[NYC];
  const int st = S.row_step();
#pragma unroll
  for (int k = 0; k < NXC; ++k) col[k] = S.col(x0 + clampi(rec[k], -(W + 1), W + 1));
#pragma unroll
  for (int i = 0; i < NYC; ++i) {
    rc[i] = S.row_coord(y0 + clampi(rec[3 + i], -(H + 1), H + 1));
    wy[i][0] = f[6 + 2 * i];
    wy[i][1] = f[7 + 2 * i];
#pragma unroll
    for (int k = 0; k < NXC; ++k) {
      cw[i][k][0] = f[12 + (i * 3 + k) * 2];
      cw[i][k][1] = f[13 + (i * 3 + k) * 2];
    }
  }
  auto row = [&](int i, int coord, float* R) {
    const typename Src::Row rr = S.row(coord);
#pragma unroll
    for (int q = 0; q < kQ; ++q) R[q] = 0.f;
#pragma unroll
    for (int k = 0; k < NXC; ++k) {
      float v[kQ + 1];
      S.run4(rr, col[k], v);
#pragma unroll
      for (int q = 0; q < kQ; ++q) R[q] = fmaf(cw[i][k][0], v[q], fmaf(cw[i][k][1], v[q + 1], R[q]));
    }
  };
  float Rc[NYC][kQ];
#pragma unroll
  for (int i = 0; i < NYC; ++i) row(i, rc[i], Rc[i]);
#pragma unroll
  for (int s = 0; s < SEG; ++s) {
    if (kFull || y0 + s < y1) {
      float o[kQ];
#pragma unroll
      for (int q = 0; q < kQ; ++q) o[q] = 0.f;
#pragma unroll
      for (int i = 0; i < NYC; ++i) {
        float Rn[kQ];
        row(i, rc[i] + (s + 1) * st, Rn);
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          o[q] = fmaf(wy[i][0], Rc[i][q], fmaf(wy[i][1], Rn[q], o[q]));
          Rc[i][q] = Rn[q];
        }
      }
      emit.template put<kFull>(s, o);
    }
  }
}

// Forward of split boxes, table in LDS: as k_box_fwd_lds (a wave per box,
// whole items of 3 columns x SEG rows), each item walking its box's shared
// corners.
template <typename OutT, int SEG, int NXC, int NYC, int kPitch, bool kTail>
__global__ __launch_bounds__(256) void k_box_fwd_lds_split(const float* __restrict__ x, const int* __restrict__ rec,
                                                           OutT* __restrict__ y, int C, int H, int W, int B, int bpg,
                                                           int per_box_p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  float* S = reinterpret_cast<float*>(smem_raw);
  const int pitch = kPitch > 0 ? kPitch : lds_pitch_dev(W);
  const int ngrp = (B + bpg - 1) / bpg;
  const int map = blockIdx.x / ngrp, grp = blockIdx.x - map * ngrp, c = map % C;
  const float* src = x + (size_t)map * H * W;
  if constexpr (kPitch > 0) {
    table_zero_edges(S, H, pitch);
    build_table_bands<float, 16, band_cols(kPitch)>(src, S, S + (H + 1) * pitch, H, W, pitch, 0.f, false);
  } else {
    build_table_lds(src, S, H, W, pitch, 0.f, false);
  }
  const LdsTable<float> tab{S, pitch, W, H};
  const int b0 = grp * bpg, nb = min(bpg, B - b0);
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG, per_box = nch * nseg;
  for (int it = threadIdx.x; it < nb * per_box_p; it += blockDim.x) {
    const int bl = __builtin_amdgcn_readfirstlane(it / per_box_p);
    const int r = it - bl * per_box_p;
    if (r >= per_box) continue;
    const ItemPos<SEG, kQ> ip(r, nch, H, W, kTail);
    const int b = b0 + bl;
    const int* rb = rec + (size_t)(c * B + b) * 32;
    OutT* out = y + ((size_t)map * B + b) * H * W;
    StoreRows<OutT, float> em{out, W, ip.x0, ip.y0 * W + ip.x0};
    corner_walk<SEG, NXC, NYC, !kTail>(tab, rb, ip.x0, ip.y0, min(ip.y0 + SEG, H), em);
  }
}

// Adjoint corner records of split boxes for the backward, 32 words per box.
// The transpose of a split box's correlation is the mirrored split box: column
// corners k' = 1 - (b, m, a), row corners r' = 1 - (d, n, c) (ascending), and
// mirrored piece (i', j') carries w(ny-1-i', nx-1-j').  Each mirrored corner
// is split as e = f + alpha with alpha in (0, 1] (f = ceil(e) - 1), so that
// the column (row) difference across a corner is the one-sided derivative the
// box gradient takes.  Words: 0..2 column floors, 3..5 row floors, 6..8
// alpha, 9..11 beta, 12..20 coef'(ri, kj) of the mirrored pieces (as in the
// forward corner record); fp64 edges, each word rounded once.
__global__ void k_box_prep_corners_adj(const float* __restrict__ boxes, const float* __restrict__ piece_w, int CB,
                                       int nx, int ny, int* __restrict__ table) {
  const int box = blockIdx.x * blockDim.x + threadIdx.x;
  if (box >= CB) return;
  const float* q = boxes + (size_t)box * 4;
  const double cx = q[0], cy = q[1], rx = q[2], ry = q[3];
  const double a = 0.5 + cx - rx, b = 0.5 + cx + rx, c = 0.5 + cy - ry, d = 0.5 + cy + ry;
  const double ke[3] = {1.0 - b, nx == 2 ? 1.0 - (a + b) / 2 : 1.0 - a, 1.0 - a};
  const double re[3] = {1.0 - d, ny == 2 ? 1.0 - (c + d) / 2 : 1.0 - c, 1.0 - c};
  const float* wp = piece_w + (size_t)box * nx * ny;
  auto w = [&](int i, int j) -> double {  // weight of mirrored piece (i, j)
    return (i < 0 || j < 0 || i >= ny || j >= nx) ? 0.0 : (double)wp[(ny - 1 - i) * nx + (nx - 1 - j)];
  };
  int* r = table + (size_t)box * 32;
  float* f = reinterpret_cast<float*>(r);
  for (int k = 0; k <= nx; ++k) {
    int fl;
    double al;
    edge_split_upper(ke[k], 1 << 20, fl, al);
    r[k] = fl;
    f[6 + k] = (float)al;
  }
  for (int i = 0; i <= ny; ++i) {
    int fl;
    double be;
    edge_split_upper(re[i], 1 << 20, fl, be);
    r[3 + i] = fl;
    f[9 + i] = (float)be;
    for (int k = 0; k <= nx; ++k) f[12 + i * 3 + k] = (float)(w(i - 1, k - 1) - w(i - 1, k) - w(i, k - 1) + w(i, k));
  }
  for (int k = 21; k < 32; ++k) r[k] = 0;
}

// Backward walk of one split box over its mirrored corners on the table of
// an upstream-gradient map (record above).  For a table row R read at step s
// for row corner ri (R = y0 + s + f_ri + 1; R = y0 + f_ri at the start) and
// column corner kj, with D = S(R, x+f_kj+1) - S(R, x+f_kj) and X = S(R,
// x+f_kj) + alpha_kj * D (the row interpolated at the corner):
//   input gradient: acc[s'][q] += coef(ri, kj) * wy * X for the output rows
//     s' that read R (wy = beta for the row below the corner, 1 - beta for
//     the row above);
//   per-tap-row sums for the parameter gradient, with the input values v:
//     PX[ri][t][kj] += v[s'] * X and PD[ri][t][kj] += v[s'] * D, t = 1 for
//     the output row s' = s (R = its row f + 1), t = 0 for s' = s + 1.
template <int SEG, int NXC, int NYC, typename Src>
__device__ __forceinline__ void corner_adjoint_walk(const Src& S, const int* __restrict__ rec, int x0, int y0,
                                                    const float (&v)[SEG][kQ], float (&acc)[SEG][kQ],
                                                    float (&PX)[NYC][2][NXC], float (&PD)[NYC][2][NXC]) {
  const float* f = reinterpret_cast<const float*>(rec);
  const int W = S.W, H = S.H;
  const int st = S.row_step();
  typename Src::Col col[NXC];
  float al[NXC];
#pragma unroll
  for (int k = 0; k < NXC; ++k) {
    col[k] = S.col(x0 + clampi(rec[k], -(W + 1), W + 1));
    al[k] = f[6 + k];
  }
#pragma unroll
  for (int i = 0; i < NYC; ++i) {
    const int r0 = S.row_coord(y0 + clampi(rec[3 + i], -(H + 1), H + 1));
    const float be = f[9 + i], wy0 = 1.f - be;
    float cf[NXC];
#pragma unroll
    for (int k = 0; k < NXC; ++k) cf[k] = f[12 + i * 3 + k];
    // step s = -1 reads row y0 + f (the upper row of output row 0); step s
    // reads row y0 + s + f + 1 (lower row of output s, upper row of s + 1)
#pragma unroll
    for (int s = -1; s < SEG; ++s) {
      const typename Src::Row rr = S.row(r0 + (s + 1) * st);
      float R[kQ] = {0.f, 0.f, 0.f};
#pragma unroll
      for (int k = 0; k < NXC; ++k) {
        float t[kQ + 1];
        S.run4(rr, col[k], t);
#pragma unroll
        for (int q = 0; q < kQ; ++q) {
          const float D = t[q + 1] - t[q];
          const float X = fmaf(al[k], D, t[q]);
          R[q] = fmaf(cf[k], X, R[q]);
          if (s >= 0) {
            PX[i][1][k] = fmaf(v[s][q], X, PX[i][1][k]);
            PD[i][1][k] = fmaf(v[s][q], D, PD[i][1][k]);
          }
          if (s + 1 < SEG) {
            PX[i][0][k] = fmaf(v[s + 1][q], X, PX[i][0][k]);
            PD[i][0][k] = fmaf(v[s + 1][q], D, PD[i][0][k]);
          }
        }
      }
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        if (s >= 0) acc[s][q] = fmaf(be, R[q], acc[s][q]);
        if (s + 1 < SEG) acc[s + 1][q] = fmaf(wy0, R[q], acc[s + 1][q]);
      }
    }
  }
}

// One item's share of a split box's gradients from its per-tap-row sums
// (adjoint corner record f): per mirrored corner (ri, kj),
// Q = (1-beta) PX0 + beta PX1 (the corner's lookup, weighted by x),
// QX = (1-beta) PD0 + beta PD1 (its x derivative), QY = PX1 - PX0 (its y
// derivative); then
//   dL/dk'_kj = sum_ri coef(ri, kj) QX,  dL/dr'_ri = sum_kj coef(ri, kj) QY,
//   dL/dw'(i, j) = Q(i+1, j+1) - Q(i+1, j) - Q(i, j+1) + Q(i, j)
// (the mirrored piece's adjoint sum weighted by x).  Mirroring back:
// dL/dk_j = -dL/dk'_{nx-j}, a cut edge (the mean of the outer two) gives half
// to each, and dL/dw(i, j) = dL/dw'(ny-1-i, nx-1-j).  g8 = (dL/da, dL/db,
// dL/dc, dL/dd, dL/dw_0 .. dL/dw_3), unused weight slots 0.
template <int NXC, int NYC>
__device__ __forceinline__ void split_box_grads(const float* __restrict__ f, const float (&PX)[NYC][2][NXC],
                                                const float (&PD)[NYC][2][NXC], float (&g8)[8]) {
  constexpr int nx = NXC - 1, ny = NYC - 1;
  float Q[NYC][NXC], gk[NXC], gr[NYC];
#pragma unroll
  for (int k = 0; k < NXC; ++k) gk[k] = 0.f;
#pragma unroll
  for (int i = 0; i < NYC; ++i) {
    const float be = f[9 + i], wy0 = 1.f - be;
    gr[i] = 0.f;
#pragma unroll
    for (int k = 0; k < NXC; ++k) {
      const float cf = f[12 + i * 3 + k];
      Q[i][k] = fmaf(wy0, PX[i][0][k], be * PX[i][1][k]);
      gk[k] = fmaf(cf, fmaf(wy0, PD[i][0][k], be * PD[i][1][k]), gk[k]);
      gr[i] = fmaf(cf, PX[i][1][k] - PX[i][0][k], gr[i]);
    }
  }
  // mirrored corner kj is original corner nx - kj, with the sign flipped
  g8[0] = -gk[nx] - (nx == 2 ? 0.5f * gk[1] : 0.f);
  g8[1] = -gk[0] - (nx == 2 ? 0.5f * gk[1] : 0.f);
  g8[2] = -gr[ny] - (ny == 2 ? 0.5f * gr[1] : 0.f);
  g8[3] = -gr[0] - (ny == 2 ? 0.5f * gr[1] : 0.f);
#pragma unroll
  for (int k = 4; k < 8; ++k) g8[k] = 0.f;
#pragma unroll
  for (int i = 0; i < ny; ++i)
#pragma unroll
    for (int j = 0; j < nx; ++j)
      g8[4 + (ny - 1 - i) * nx + (nx - 1 - j)] = (Q[i + 1][j + 1] - Q[i + 1][j]) - (Q[i][j + 1] - Q[i][j]);
}

// Backward of split boxes, table in LDS: as k_box_bwd_lds (one block per map,
// one item of 3 columns x SEG rows per thread, input values in registers), one
// walk over each box's mirrored corners.  Each wave writes its split_box_grads
// sums to partials[(n * nw + wave) * C*B + c*B + b][8].
// kPitch > 0: the table's row pitch compiled in and its column sums formed in
// registers, as in k_box_bwd_lds.
template <int SEG, int NXC, int NYC, int kMaxT, int kPitch>
__global__ __launch_bounds__(kMaxT) void k_box_bwd_lds_split(const float* __restrict__ x, const int* __restrict__ rec,
                                                           const float* __restrict__ gy, float* __restrict__ gx,
                                                           float* __restrict__ partials, int C, int H, int W,
                                                           int B) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int pitch = kPitch > 0 ? kPitch : lds_pitch_dev(W);
  float* SG = reinterpret_cast<float*>(smem_raw);
  const int map = blockIdx.x, n = map / C, c = map - n * C;
  const int nw = blockDim.x >> 6, wave = threadIdx.x >> 6;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const int it = threadIdx.x;
  const bool active = it < nch * nseg;
  const int seg = it / nch, ch = it - seg * nch;
  const int x0 = ch * kQ, y0 = seg * SEG;
  const size_t plane = (size_t)H * W;
  const float* g0 = gy + (size_t)map * B * plane;
  float v[SEG][kQ], acc[SEG][kQ];
  load_item<SEG>(x + (size_t)map * plane, H, W, x0, y0, active, v);
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[s][q] = 0.f;
  const LdsTable<float> tg{SG, pitch, W, H};
  // rows per band: 8-row items have fewer waves to a map, and with one column a
  // lane the registers for 32 rows in flight
  constexpr int kRows = SEG == 8 && band_cols(kPitch) == 1 ? 32 : 16;
  if constexpr (kPitch > 0) table_zero_edges(SG, H, pitch);
  for (int b = 0; b < B; ++b) {
    if constexpr (kPitch > 0) {
      build_table_bands<float, kRows, band_cols(kPitch)>(
          g0 + b * plane, SG, SG + (H + 1) * pitch, H, W, pitch, 0.f, false);
    } else {
      __syncthreads();
      build_table_lds(g0 + b * plane, SG, H, W, pitch, 0.f, false);
    }
    const int cb = c * B + b;
    const int* rb = rec + (size_t)cb * 32;
    float PX[NYC][2][NXC], PD[NYC][2][NXC];
#pragma unroll
    for (int i = 0; i < NYC; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < NXC; ++k) { PX[i][t][k] = 0.f; PD[i][t][k] = 0.f; }
    if (active) corner_adjoint_walk<SEG, NXC, NYC>(tg, rb, x0, y0, v, acc, PX, PD);
    float g8[8];
    split_box_grads<NXC, NYC>(reinterpret_cast<const float*>(rb), PX, PD, g8);
    float* pp = partials + (((size_t)n * nw + wave) * C * B + cb) * 8;
    store_wave_partial(g8, pp);
    store_wave_partial(g8 + 4, pp + 4);
  }
  if (active && gx != nullptr) store_item<SEG>(gx + (size_t)map * plane, H, W, x0, y0, acc);
}

// Forward of split boxes, table in HBM: as k_box_fwd_gather (one block per
// (map, box, block of 256 items), one map's blocks on one XCD).
template <typename OutT, int SEG, int NXC, int NYC, bool kNT>
__global__ __launch_bounds__(256) void k_box_fwd_gather_split(const float* __restrict__ sat,
                                                              const int* __restrict__ rec, OutT* __restrict__ y,
                                                              int C, int H, int W, int B, int nblk, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int blk = L % nblk, mb = L / nblk;
  const int b = mb % B, map = mb / B, c = map % C;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const int it = blk * 256 + threadIdx.x;
  if (it >= nch * nseg) return;
  const int seg = it / nch, ch = it - seg * nch;
  const GlobalTable<float, true> tab{sat + (size_t)map * (H + 1) * (W + 1), W + 1, W, H};
  const int* rb = rec + (size_t)(c * B + b) * 32;
  OutT* out = y + ((size_t)map * B + b) * H * W;
  const int x0 = ch * kQ, y0 = seg * SEG, y1 = min(y0 + SEG, H);
  StoreRows<OutT, float, kNT> em{out, W, x0, y0 * W + x0};
  if (y0 + SEG <= H && x0 + kQ <= W) corner_walk<SEG, NXC, NYC, true>(tab, rb, x0, y0, y1, em);
  else corner_walk<SEG, NXC, NYC, false>(tab, rb, x0, y0, y1, em);
}

// Backward of split boxes, tables of the upstream-gradient maps in HBM: as
// k_box_bwd_gather (one block per (map, block of 256 items), looping over the
// boxes).  Each wave writes its split_box_grads sums to
// partials[((n * nblk + blk) * 4 + wave) * C*B + c*B + b][8].
template <int SEG, int NXC, int NYC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_box_bwd_gather_split(
    const float* __restrict__ x, const float* __restrict__ sat_g, const int* __restrict__ rec,
    float* __restrict__ gx, float* __restrict__ partials, int C, int H, int W, int B, int nblk, int total) {
  const int L = xcd_remap(blockIdx.x, gridDim.x);
  if (L >= total) return;
  const int blk = L % nblk, map = L / nblk;
  const int n = map / C, c = map - n * C;
  const int wave = threadIdx.x >> 6;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const int it = blk * 256 + threadIdx.x;
  const bool active = it < nch * nseg;
  const int seg = it / nch, ch = it - seg * nch;
  const int x0 = ch * kQ, y0 = seg * SEG;
  const size_t tsz = (size_t)(H + 1) * (W + 1);
  float v[SEG][kQ], acc[SEG][kQ];
  load_item<SEG>(x + (size_t)map * H * W, H, W, x0, y0, active, v);
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[s][q] = 0.f;
  for (int b = 0; b < B; ++b) {
    const GlobalTable<float> tg{sat_g + ((size_t)map * B + b) * tsz, W + 1, W, H};
    const int cb = c * B + b;
    const int* rb = rec + (size_t)cb * 32;
    float PX[NYC][2][NXC], PD[NYC][2][NXC];
#pragma unroll
    for (int i = 0; i < NYC; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < NXC; ++k) { PX[i][t][k] = 0.f; PD[i][t][k] = 0.f; }
    if (active) corner_adjoint_walk<SEG, NXC, NYC>(tg, rb, x0, y0, v, acc, PX, PD);
    float g8[8];
    split_box_grads<NXC, NYC>(reinterpret_cast<const float*>(rb), PX, PD, g8);
    float* pp = partials + ((((size_t)n * nblk + blk) * 4 + wave) * C * B + cb) * 8;
    store_wave_partial(g8, pp);
    store_wave_partial(g8 + 4, pp + 4);
  }
  if (active && gx != nullptr) store_item<SEG>(gx + (size_t)map * H * W, H, W, x0, y0, acc);
}

// Fixed-tree sum of the split partials [Pn][CB][8] (as k_box_grad_reduce) and
// the change of variables of the box edges; the weight gradients as summed.
__global__ __launch_bounds__(256) void k_split_grad_reduce(const float* __restrict__ partials, int Pn, int CB,
                                                           int P, float* __restrict__ grad_boxes,
                                                           float* __restrict__ grad_w) {
  __shared__ float4 red[4][kReduceBoxes][2];
  const int j = threadIdx.x % kReduceBoxes, q = threadIdx.x / kReduceBoxes;
  const int i = blockIdx.x * kReduceBoxes + j;
  float4 s0 = make_float4(0.f, 0.f, 0.f, 0.f), s1 = s0;
  if (i < CB)
    for (int p = q; p < Pn; p += 256 / kReduceBoxes) {
      const float4* v = reinterpret_cast<const float4*>(partials + ((size_t)p * CB + i) * 8);
      const float4 a = v[0], b = v[1];
      s0.x += a.x; s0.y += a.y; s0.z += a.z; s0.w += a.w;
      s1.x += b.x; s1.y += b.y; s1.z += b.z; s1.w += b.w;
    }
#pragma unroll
  for (int m = 16; m < 64; m <<= 1) {
    s0.x += __shfl_xor(s0.x, m); s0.y += __shfl_xor(s0.y, m); s0.z += __shfl_xor(s0.z, m); s0.w += __shfl_xor(s0.w, m);
    s1.x += __shfl_xor(s1.x, m); s1.y += __shfl_xor(s1.y, m); s1.z += __shfl_xor(s1.z, m); s1.w += __shfl_xor(s1.w, m);
  }
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) < kReduceBoxes) { red[wave][j][0] = s0; red[wave][j][1] = s1; }
  __syncthreads();
  if (threadIdx.x < kReduceBoxes && i < CB) {
    float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float4 a = red[w][j][0], b = red[w][j][1];
      t[0] += a.x; t[1] += a.y; t[2] += a.z; t[3] += a.w;
      t[4] += b.x; t[5] += b.y; t[6] += b.z; t[7] += b.w;
    }
    if (grad_boxes)
      *reinterpret_cast<float4*>(grad_boxes + (size_t)i * 4) = make_float4(t[0] + t[1], t[2] + t[3], t[1] - t[0], t[3] - t[2]);
    if (grad_w)
      for (int k = 0; k < P; ++k) grad_w[(size_t)i * P + k] = t[4 + k];
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_box_prep_corners(const float* boxes, const float* piece_w, int C, int B, int nx, int ny,
                                   void* table, hipStream_t s) {
  const int n = C * B;
  hipLaunchKernelGGL(k_box_prep_corners, dim3((n + 255) / 256), dim3(256), 0, s, boxes, piece_w, n, nx, ny,
                     (int*)table);
  return last_error();
}

// Narrow maps of several strips of bands are staged, as for whole boxes, in calls
// of four waves per CU and more: two strips where one wave walks them alone, three
// elsewhere (backward of 2 x 3141 maps of 86x8, 8 boxes 324 us from registers, 227
// staged; 6 x 519 of 50x24, 8 boxes 149 and 122; two waves and two strips, 8 x 512
// of 100x22, 4 boxes 147 and 164; forward of 10 x 598 of 80x12 57 and 44).
static bool split_staged(int W, int H, int waves, long blocks) {
  return W <= 24 && H > waves * (waves == 1 ? 32 : 64) && blocks * waves >= 1024;
}

template <typename OutT, int NXC, int NYC>
static void fwd_split_t(const float* x, const int* rec, void* y, int N, int C, int H, int W, int B, hipStream_t s) {
  constexpr int SEG = 16;
  const FwdGeom g = fwd_geom_items(N, C, B, n_chunks(W) * n_segs(H, SEG), 256);
  const bool tail = W < kQ || H < SEG;
  const int pc = tail || split_staged(W, H, g.threads / 64, (long)N * C * g.ngrp) ? 0 : lds_pitch_class(H, W);
  const size_t shm = table_lds_bytes(H, W, pc, g.threads);
  auto go = [&](auto kp, auto kt) {
    hipLaunchKernelGGL((k_box_fwd_lds_split<OutT, SEG, NXC, NYC, decltype(kp)::value, decltype(kt)::value>),
                       dim3(N * C * g.ngrp), dim3(g.threads), shm, s, x, rec, (OutT*)y, C, H, W, B, g.bpg, g.per_box_p);
  };
  if (tail) go(std::integral_constant<int, 0>{}, std::true_type{});
  else with_pitch(pc, [&](auto kp) { go(kp, std::false_type{}); });
}

template <typename OutT>
static void fwd_split_mode(const float* x, const int* rec, void* y, int N, int C, int H, int W, int B, int nx, int ny,
                           hipStream_t s) {
  if (nx == 2 && ny == 2) fwd_split_t<OutT, 3, 3>(x, rec, y, N, C, H, W, B, s);
  else if (nx == 2) fwd_split_t<OutT, 3, 2>(x, rec, y, N, C, H, W, B, s);
  else fwd_split_t<OutT, 2, 3>(x, rec, y, N, C, H, W, B, s);
}

hipError_t launch_box_fwd_lds_split(const float* x, const int* rec, void* y, bool bf16_out, int N, int C, int H, int W,
                                    int B, int nx, int ny, hipStream_t s) {
  if (bf16_out) fwd_split_mode<uint16_t>(x, rec, y, N, C, H, W, B, nx, ny, s);
  else fwd_split_mode<float>(x, rec, y, N, C, H, W, B, nx, ny, s);
  return last_error();
}

hipError_t launch_box_prep_corners_adj(const float* boxes, const float* piece_w, int C, int B, int nx, int ny,
                                       void* table, hipStream_t s) {
  const int n = C * B;
  hipLaunchKernelGGL(k_box_prep_corners_adj, dim3((n + 255) / 256), dim3(256), 0, s, boxes, piece_w, n, nx, ny,
                     (int*)table);
  return last_error();
}

template <int SEG, int NXC, int NYC, int kMaxT>
static void bwd_split_t(const float* x, const int* rec, const float* gy, float* gx, float* partials, int N, int C,
                        int H, int W, int B, hipStream_t s) {
  const int threads = ((n_chunks(W) * n_segs(H, SEG) + 63) / 64) * 64;
  const int pc = SEG == 8 && split_staged(W, H, threads / 64, (long)N * C) ? 0 : lds_pitch_class(H, W);
  const size_t shm = table_lds_bytes(H, W, pc, threads);
  with_pitch(pc, [&](auto kp) {
    hipLaunchKernelGGL((k_box_bwd_lds_split<SEG, NXC, NYC, kMaxT, decltype(kp)::value>), dim3(N * C), dim3(threads),
                       shm, s, x, rec, gy, gx, partials, C, H, W, B);
  });
}

template <int SEG, int kMaxT>
static void bwd_split_mode(const float* x, const int* rec, const float* gy, float* gx, float* partials, int N, int C,
                           int H, int W, int B, int nx, int ny, hipStream_t s) {
  if (nx == 2 && ny == 2) bwd_split_t<SEG, 3, 3, kMaxT>(x, rec, gy, gx, partials, N, C, H, W, B, s);
  else if (nx == 2) bwd_split_t<SEG, 3, 2, kMaxT>(x, rec, gy, gx, partials, N, C, H, W, B, s);
  else bwd_split_t<SEG, 2, 3, kMaxT>(x, rec, gy, gx, partials, N, C, H, W, B, s);
}

// As the whole-box backward: 8-row items in blocks of up to 256 threads, else
// 4-row items (at most 107 VGPRs) in blocks of up to kBwdLdsItems threads.
hipError_t launch_box_bwd_lds_split(const float* x, const int* rec, const float* gy, float* gx, float* partials, int N,
                                    int C, int H, int W, int B, int nx, int ny, hipStream_t s) {
  const int seg = box_bwd_lds_seg(H, W, kBwdLdsItems);
  if (seg == 8) bwd_split_mode<8, 256>(x, rec, gy, gx, partials, N, C, H, W, B, nx, ny, s);
  else if (seg == 4 && n_chunks(W) * n_segs(H, 4) <= 256)
    bwd_split_mode<4, 256>(x, rec, gy, gx, partials, N, C, H, W, B, nx, ny, s);
  else if (seg == 4) bwd_split_mode<4, kBwdLdsItems>(x, rec, gy, gx, partials, N, C, H, W, B, nx, ny, s);
  else return hipErrorInvalidValue;
  return last_error();
}

template <typename OutT, int NXC, int NYC>
static void fwd_gather_split_t(const float* sat, const int* rec, void* y, int N, int C, int H, int W, int B,
                               hipStream_t s) {
  constexpr int SEG = 16;
  const int nblk = (n_chunks(W) * n_segs(H, SEG) + 255) / 256;
  const int total = N * C * B * nblk;
  with_flag(stream_out((size_t)N * C * B * H * W, sizeof(OutT)), [&](auto kn) {
    hipLaunchKernelGGL((k_box_fwd_gather_split<OutT, SEG, NXC, NYC, decltype(kn)::value>), dim3(pad8(total)),
                       dim3(256), 0, s, sat, rec, (OutT*)y, C, H, W, B, nblk, total);
  });
}

template <typename OutT>
static void fwd_gather_split_mode(const float* sat, const int* rec, void* y, int N, int C, int H, int W, int B, int nx,
                                  int ny, hipStream_t s) {
  if (nx == 2 && ny == 2) fwd_gather_split_t<OutT, 3, 3>(sat, rec, y, N, C, H, W, B, s);
  else if (nx == 2) fwd_gather_split_t<OutT, 3, 2>(sat, rec, y, N, C, H, W, B, s);
  else fwd_gather_split_t<OutT, 2, 3>(sat, rec, y, N, C, H, W, B, s);
}

hipError_t launch_box_fwd_gather_split(const float* sat, const int* rec, void* y, bool bf16_out, int N, int C, int H,
                                       int W, int B, int nx, int ny, hipStream_t s) {
  if (bf16_out) fwd_gather_split_mode<uint16_t>(sat, rec, y, N, C, H, W, B, nx, ny, s);
  else fwd_gather_split_mode<float>(sat, rec, y, N, C, H, W, B, nx, ny, s);
  return last_error();
}

template <int NXC, int NYC>
static void bwd_gather_split_t(const float* x, const float* sat_g, const int* rec, float* gx, float* partials, int N,
                               int C, int H, int W, int B, hipStream_t s) {
  const int nblk = box_bwd_gather_blocks(H, W);
  const int total = N * C * nblk;
  hipLaunchKernelGGL((k_box_bwd_gather_split<kBwdGatherSeg, NXC, NYC>), dim3(pad8(total)), dim3(256), 0, s, x, sat_g,
                     rec, gx, partials, C, H, W, B, nblk, total);
}

hipError_t launch_box_bwd_gather_split(const float* x, const float* sat_g, const int* rec, float* gx, float* partials,
                                       int N, int C, int H, int W, int B, int nx, int ny, hipStream_t s) {
  if (nx == 2 && ny == 2) bwd_gather_split_t<3, 3>(x, sat_g, rec, gx, partials, N, C, H, W, B, s);
  else if (nx == 2) bwd_gather_split_t<3, 2>(x, sat_g, rec, gx, partials, N, C, H, W, B, s);
  else bwd_gather_split_t<2, 3>(x, sat_g, rec, gx, partials, N, C, H, W, B, s);
  return last_error();
}

hipError_t launch_split_grad_reduce(const float* partials, int Pn, int CB, int P, float* grad_boxes, float* grad_w,
                                    hipStream_t s) {
  hipLaunchKernelGGL(k_split_grad_reduce, dim3((CB + kReduceBoxes - 1) / kReduceBoxes), dim3(256), 0, s, partials,
                     Pn, CB, P, grad_boxes, grad_w);
  return last_error();
}

}  // namespace bc
