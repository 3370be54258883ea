// Device code shared by the box filter kernels (tables in LDS, walks over a
// table, item loads and stores) and their launch geometry.  gfx950, wave64.
#pragma once
#include "bc_common.hpp"
#include "bc_internal.hpp"

#include <type_traits>

namespace bc {

// ---------------------------------------------------------------------------
// Helpers
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lds_pitch_dev(int W) { return (W + 7) | 1; }

template <typename OutT, typename T> __device__ __forceinline__ OutT convert_out(T v);
template <> __device__ __forceinline__ float convert_out<float, float>(float v) { return v; }
template <> __device__ __forceinline__ int convert_out<int, int>(int v) { return v; }
template <> __device__ __forceinline__ uint16_t convert_out<uint16_t, float>(float v) {
  return __builtin_bit_cast(uint16_t, (__bf16)v);  // round to nearest even (v_cvt_pk_bf16_f32)
}

// Grid-to-work mapping that keeps consecutive logical blocks on one XCD.
// Blocks are dispatched to the 8 XCDs round-robin by block index; logical
// block L = xcd * (grid/8) + slot gives each XCD one contiguous range of
// logical blocks, so all blocks reading one map's table share that XCD's L2.
// The grid is padded to a multiple of 8; logical ids >= total exit.
__device__ __forceinline__ int xcd_remap(int bid, int grid) {
  const int per = grid >> 3;
  return (bid & 7) * per + (bid >> 3);
}
inline int pad8(int n) { return (n + 7) & ~7; }

// Mean of one map, fp32, fixed summation order for a given block size.
__device__ inline float block_mean(const float* __restrict__ src, int n, float* red) {
  float s = 0.f;
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += src[i];
  s = wave_sum(s);
  const int wave = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  if ((threadIdx.x & 63) == 0) red[wave] = s;
  __syncthreads();
  float tot = 0.f;
  for (int w = 0; w < nw; ++w) tot += red[w];
  __syncthreads();
  return tot / (float)n;
}

// 16-byte vector of the map element type.
template <typename T> struct Vec4;
template <> struct Vec4<float> { using type = float4; };
template <> struct Vec4<int> { using type = int4; };

// Zero row 0 and columns -kPad..0 of every row of a padded LDS table.
template <typename T>
__device__ __forceinline__ void table_zero_edges(T* S, int H, int pitch) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int v = tid; v < pitch; v += nt) S[v] = (T)0;
  for (int k = tid; k < H * (kPad + 1); k += nt) {
    const int u = 1 + k / (kPad + 1);
    S[u * pitch + k - (u - 1) * (kPad + 1)] = (T)0;
  }
}

// Row pass of a padded LDS table whose interior holds column prefix sums:
// lanes own rows, reading kScan elements ahead before writing, so that a
// lane's LDS reads overlap; also fills the right padding.
template <typename T>
__device__ __forceinline__ void table_row_pass(T* S, int H, int W, int pitch) {
  constexpr int kScan = 16;
  T* R = S + kPad;
  for (int u = threadIdx.x + 1; u <= H; u += blockDim.x) {
    T* row = R + u * pitch;
    T run = (T)0;
    int v = 1;
    for (; v + kScan - 1 <= W; v += kScan) {
      T r[kScan];
#pragma unroll
      for (int k = 0; k < kScan; ++k) r[k] = row[v + k];
#pragma unroll
      for (int k = 0; k < kScan; ++k) {
        run += r[k];
        row[v + k] = run;
      }
    }
    for (; v <= W; ++v) {
      run += row[v];
      row[v] = run;
    }
#pragma unroll
    for (int k = 1; k <= kPad; ++k) row[W + k] = run;
  }
}

// Column pass (lanes own columns) and row pass of a padded LDS table whose
// interior holds the map, each reading kScan elements ahead before it writes.
template <typename T>
__device__ __forceinline__ void table_scans(T* S, int H, int W, int pitch) {
  constexpr int kScan = 16;
  const int tid = threadIdx.x, nt = blockDim.x;
  T* R = S + kPad;
  for (int v = tid + 1; v <= W; v += nt) {
    T run = (T)0;
    int u = 1;
    for (; u + kScan - 1 <= H; u += kScan) {
      T r[kScan];
#pragma unroll
      for (int k = 0; k < kScan; ++k) r[k] = R[(u + k) * pitch + v];
#pragma unroll
      for (int k = 0; k < kScan; ++k) {
        run += r[k];
        R[(u + k) * pitch + v] = run;
      }
    }
    for (; u <= H; ++u) {
      run += R[u * pitch + v];
      R[u * pitch + v] = run;
    }
  }
  __syncthreads();
  table_row_pass(S, H, W, pitch);
  __syncthreads();
}

// Map loads that stream (each map is read once per call) are non-temporal:
// they leave the caches to the outputs the next call reads (the box
// forward's filtered maps stay cached for the mix; pose-layer step 0.627 ->
// 0.614 ms).
template <typename T>
__device__ __forceinline__ typename Vec4<T>::type load_stream4(const typename Vec4<T>::type* p) {
  typedef T v4 __attribute__((ext_vector_type(4)));
  const v4 t = __builtin_nontemporal_load(reinterpret_cast<const v4*>(p));
  typename Vec4<T>::type r;
  r.x = t.x; r.y = t.y; r.z = t.z; r.w = t.w;
  return r;
}

// Exclusive table of one H x W map in LDS, padded (LdsTable): S(u, v) at
// S[u * pitch + kPad + v].  The map is first copied into the table's interior
// with every thread issuing 16-byte loads in batches (the loads of a batch are
// all in flight together; out-of-range slots re-read the last vector and are
// not stored, so no lane branches around a load).  Then a column pass (lanes
// own columns) and the row pass, each reading kScan elements ahead before it
// writes.  With `sub`, mu is subtracted from the tabulated values.
template <typename T, bool kSkip = false>
__device__ void build_table_lds(const T* __restrict__ src, T* S, int H, int W, int pitch, float mu, bool sub) {
  using V = typename Vec4<T>::type;
  constexpr int kBatch = 8;
  const int tid = threadIdx.x, nt = blockDim.x;
  T* R = S + kPad;
  table_zero_edges(S, H, pitch);
  // Slot k of this thread is element (vector) tid + k * nt; its row and
  // column advance by the same (nt / width, nt % width) every slot, so only
  // the first position takes a division.
  const int n = H * W;
  if ((W & 3) == 0 && ((uintptr_t)src & 15) == 0) {
    const int n4 = n >> 2, W4 = W >> 2;
    const int di = nt / W4, dj = nt - di * W4;
    int j = tid % W4;
    int o = (tid / W4 + 1) * pitch + 4 * j + 1;  // table offset of the slot's first element
    const int step = di * pitch + 4 * dj, wrap = pitch - W;
    const V* s4 = reinterpret_cast<const V*>(src);
    for (int base = 0; base < n4; base += nt * kBatch) {
      // kSkip: slots past the map for every thread of the block (the tail
      // of the last batch) issue nothing, a block-uniform test (the
      // backward keeps the unconditional form, which fits its registers)
      V q[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b)
        if (!kSkip || base + b * nt < n4) q[b] = load_stream4<T>(s4 + min(base + b * nt + tid, n4 - 1));
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        if (kSkip && base + b * nt >= n4) break;
        if (tid < n4 - base - b * nt) {
          const T w4[4] = {(T)q[b].x, (T)q[b].y, (T)q[b].z, (T)q[b].w};
#pragma unroll
          for (int t = 0; t < 4; ++t) R[o + t] = sub ? (T)((float)w4[t] - mu) : w4[t];
        }
        o += step;
        j += dj;
        if (j >= W4) { j -= W4; o += wrap; }
      }
    }
  } else {
    const int di = nt / W, dj = nt - di * W;
    int i = tid / W, j = tid - i * W;
    for (int k = tid; k < n; k += nt) {
      const T v = __builtin_nontemporal_load(src + k);
      R[(i + 1) * pitch + j + 1] = sub ? (T)((float)v - mu) : v;
      i += di;
      j += dj;
      if (j >= W) { j -= W; ++i; }
    }
  }
  __syncthreads();
  table_scans(S, H, W, pitch);
}

// Table of a zero-upsampled fp32 map (the transpose of sampling every s-th
// pixel): src (Ho x Wo) placed at (s*i, s*j) of an H x W map, zeros
// elsewhere; s * (Ho - 1) < H and s * (Wo - 1) < W.  Each source value
// writes its whole s x s block of the interior (the value at the block's
// corner, zeros elsewhere), so every interior element is written once; the
// loads of a batch are in flight together.
__device__ inline void build_table_lds_up(const float* __restrict__ src, float* S, int H, int W, int pitch, int s, int Ho,
                                   int Wo) {
  constexpr int kB = 8;
  const int tid = threadIdx.x, nt = blockDim.x, n = Ho * Wo;
  float* R = S + kPad;
  table_zero_edges(S, H, pitch);
  for (int base = 0; base < n; base += nt * kB) {
    float g[kB];
#pragma unroll
    for (int b = 0; b < kB; ++b) g[b] = src[min(base + b * nt + tid, n - 1)];
#pragma unroll
    for (int b = 0; b < kB; ++b) {
      const int k = base + b * nt + tid;
      if (k < n) {
        const int i = k / Wo, j = k - i * Wo;
        const int u1 = min(s * i + s, H), v1 = min(s * j + s, W);
        for (int u = s * i; u < u1; ++u) {
          float* row = R + (u + 1) * pitch + 1;
          for (int v = s * j; v < v1; ++v) row[v] = (u == s * i && v == s * j) ? g[b] : 0.f;
        }
      }
    }
  }
  __syncthreads();
  table_scans(S, H, W, pitch);
}

// ---------------------------------------------------------------------------
// Walks with compile-time segment length (registers indexed statically)
// ---------------------------------------------------------------------------

// The columns of a Q-column item (Q a multiple of kQ) as Q / kQ groups of
// kQ, each with its own clamped run start: the LDS table's padding (kPad = 3
// columns a side) covers runs of kQ + 1 words only, so a wider item reads
// its runs group by group.
template <int Q, typename Src>
struct ColGroups {
  static_assert(Q % kQ == 0, "items are whole groups of kQ columns");
  static constexpr int NG = Q / kQ;
  typename Src::Cols c[NG];
  __device__ __forceinline__ ColGroups(const Src& S, int ba, int bb) {
#pragma unroll
    for (int g = 0; g < NG; ++g) c[g] = S.cols(ba + g * kQ, bb + g * kQ);
  }
  // x-interpolated row (table_row) for all Q columns
  template <typename T>
  __device__ __forceinline__ void row(const Src& S, int coord, const Taps<T>& tp, T* U) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) table_row(S, coord, c[g], tp, U + g * kQ);
  }
  // the kQ-word runs at both x edges, for all Q columns
  template <typename T>
  __device__ __forceinline__ void runs(const Src& S, int coord, T* sa, T* sb) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) S.template runs<kQ>(coord, c[g], sa + g * kQ, sb + g * kQ);
  }
};

// Forward walk: emit.put<kFull>(s, o) for s in [0, SEG) with y0 + s < y1.
// kFull: the item is known to be whole (y1 = y0 + SEG, x0 + kQ <= W), so no
// step or column is guarded and the unrolled window needs no register copies.
// Each step reads two new table rows (one per y edge) and reuses the two from
// the step before.  With kOffset the table holds the map minus mu, and
// mu * (clipped box area) is added back: the clipped area is the same tap
// combination applied to the clamped coordinates (the table of a constant
// image is mu * u * v).
template <int SEG, typename T, bool kOffset, bool kFull, int Q = kQ, typename Src, typename Emit>
__device__ __forceinline__ void box_walk(const Src& S, const Taps<T>& tp, int H, int W, int x0,
                                         int y0, int y1, float mu, Emit& emit) {
  const int ba = x0 + tp.ox[0], bb = x0 + tp.ox[2];
  const ColGroups<Q, Src> cl(S, ba, bb);
  const int st = S.row_step();
  const int rc = S.row_coord(y0 + tp.oy[0]), rd = S.row_coord(y0 + tp.oy[2]);
  T uc[Q], ud[Q];
  cl.row(S, rc, tp, uc);
  cl.row(S, rd, tp, ud);
  float ex[Q];
  if (kOffset) {
#pragma unroll
    for (int q = 0; q < Q; ++q)
      ex[q] = wsum4((float)tp.wx[0], (float)clampi(ba + q, 0, W), (float)tp.wx[1], (float)clampi(ba + q + 1, 0, W),
                    (float)tp.wx[2], (float)clampi(bb + q, 0, W), (float)tp.wx[3], (float)clampi(bb + q + 1, 0, W));
  }
#pragma unroll
  for (int s = 0; s < SEG; ++s) {
    const int y = y0 + s;
    if (kFull || y < y1) {
      T uc1[Q], ud1[Q];
      cl.row(S, rc + (s + 1) * st, tp, uc1);
      cl.row(S, rd + (s + 1) * st, tp, ud1);
      T o[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q)
        o[q] = wsum4(tp.wy[0], uc[q], tp.wy[1], uc1[q], tp.wy[2], ud[q], tp.wy[3], ud1[q]);
      if (kOffset) {
        const float ey = wsum4((float)tp.wy[0], (float)clampi(y + tp.oy[0], 0, H), (float)tp.wy[1],
                               (float)clampi(y + tp.oy[1], 0, H), (float)tp.wy[2], (float)clampi(y + tp.oy[2], 0, H),
                               (float)tp.wy[3], (float)clampi(y + tp.oy[3], 0, H));
#pragma unroll
        for (int q = 0; q < Q; ++q) o[q] = add_offset(o[q], mu, ex[q] * ey);
      }
      emit.template put<kFull>(s, o);
#pragma unroll
      for (int q = 0; q < Q; ++q) { uc[q] = uc1[q]; ud[q] = ud1[q]; }
    }
  }
}

// Walk for boxes with integer corners (make_taps_rounded records): each
// output is Eq. 2's four-corner difference with no interpolation, so per
// output row the walk reads one table row per y edge, each a run of kQ
// columns at both x edges:  o = (S(y+d, x+b) - S(y+d, x+a)) - (S(y+c, x+b) -
// S(y+c, x+a)).  emit.put<kFull>(s, o) for s in [0, SEG) with y0 + s < y1.
// With kOffset the table holds the map minus mu, and mu * (clipped area) is
// added back.
template <int SEG, typename T, bool kOffset, bool kFull, int Q = kQ, typename Src, typename Emit>
__device__ __forceinline__ void box_walk_int(const Src& S, const Taps<T>& tp, int H, int W, int x0, int y0,
                                             int y1, float mu, Emit& emit) {
  const int ba = x0 + tp.ox[0], bb = x0 + tp.ox[2];
  const ColGroups<Q, Src> cl(S, ba, bb);
  const int st = S.row_step();
  const int rc = S.row_coord(y0 + tp.oy[0]), rd = S.row_coord(y0 + tp.oy[2]);
  float ex[Q];
  if (kOffset) {
#pragma unroll
    for (int q = 0; q < Q; ++q) ex[q] = (float)(clampi(bb + q, 0, W) - clampi(ba + q, 0, W));
  }
#pragma unroll
  for (int s = 0; s < SEG; ++s) {
    const int y = y0 + s;
    if (kFull || y < y1) {
      T ca[Q], cb[Q], da[Q], db[Q];
      cl.runs(S, rc + s * st, ca, cb);
      cl.runs(S, rd + s * st, da, db);
      T o[Q];
#pragma unroll
      for (int q = 0; q < Q; ++q) o[q] = (db[q] - da[q]) - (cb[q] - ca[q]);
      if (kOffset) {
        const float ey = (float)(clampi(y + tp.oy[2], 0, H) - clampi(y + tp.oy[0], 0, H));
#pragma unroll
        for (int q = 0; q < Q; ++q) o[q] = add_offset(o[q], mu, ex[q] * ey);
      }
      emit.template put<kFull>(s, o);
    }
  }
}

// Strided forward walk of one item: output column j (input column x = s*j)
// and output rows i0 .. i1-1 (input rows s*i).  Consecutive outputs are s
// rows apart and share no table rows, so each output reads its own: two rows
// per y edge (one with integer corners), runs of two columns (one) at both x
// edges -- the 16 (4) samples of Eq. 2-3.  emit.put(k, o) for output row
// i0 + k.  With kOffset the table holds the map minus mu, and mu * (clipped
// area) is added back.
template <int SEGS, typename T, bool kOffset, bool kInt, typename Src, typename Emit>
__device__ __forceinline__ void box_walk_strided(const Src& S, const Taps<T>& tp, int H, int W, int x, int i0,
                                                 int i1, int s, float mu, Emit& emit) {
  const int ba = x + tp.ox[0], bb = x + tp.ox[2];
  const typename Src::Cols cl = S.cols(ba, bb);
  const int st = S.row_step();
  float ex = 0.f;
  if (kOffset) {
    ex = kInt ? (float)(clampi(bb, 0, W) - clampi(ba, 0, W))
              : wsum4((float)tp.wx[0], (float)clampi(ba, 0, W), (float)tp.wx[1], (float)clampi(ba + 1, 0, W),
                      (float)tp.wx[2], (float)clampi(bb, 0, W), (float)tp.wx[3], (float)clampi(bb + 1, 0, W));
  }
#pragma unroll
  for (int k = 0; k < SEGS; ++k) {
    const int i = i0 + k;
    if (i < i1) {
      const int y = s * i;
      const int rc = S.row_coord(y + tp.oy[0]), rd = S.row_coord(y + tp.oy[2]);
      T o;
      if constexpr (kInt) {
        T ca[1], cb[1], da[1], db[1];
        S.template runs<1>(rc, cl, ca, cb);
        S.template runs<1>(rd, cl, da, db);
        o = (db[0] - da[0]) - (cb[0] - ca[0]);
      } else {
        T u[4];
        const int rows[4] = {rc, rc + st, rd, rd + st};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          T sa[2], sb[2];
          S.template runs<2>(rows[r], cl, sa, sb);
          u[r] = wsum4(tp.wx[0], sa[0], tp.wx[1], sa[1], tp.wx[2], sb[0], tp.wx[3], sb[1]);
        }
        o = wsum4(tp.wy[0], u[0], tp.wy[1], u[1], tp.wy[2], u[2], tp.wy[3], u[3]);
      }
      if (kOffset) {
        const float ey = kInt ? (float)(clampi(y + tp.oy[2], 0, H) - clampi(y + tp.oy[0], 0, H))
                              : wsum4((float)tp.wy[0], (float)clampi(y + tp.oy[0], 0, H), (float)tp.wy[1],
                                      (float)clampi(y + tp.oy[1], 0, H), (float)tp.wy[2],
                                      (float)clampi(y + tp.oy[2], 0, H), (float)tp.wy[3],
                                      (float)clampi(y + tp.oy[3], 0, H));
        o = add_offset(o, mu, ex * ey);
      }
      emit.put(k, o);
    }
  }
}

// Emitter of one strided output column: output row i0 + k at plane offset
// off0 + k * Wo (off0 = i0 * Wo + j).
template <typename OutT, typename T>
struct StoreCol {
  OutT* out;
  int Wo, off0;
  __device__ __forceinline__ void put(int k, T o) { out[(unsigned)(off0 + k * Wo)] = convert_out<OutT, T>(o); }
};

// Forward walk of one item: integer-corner or interpolated.
template <int SEG, typename T, bool kOffset, bool kFull, bool kInt, int Q = kQ, typename Src, typename Emit>
__device__ __forceinline__ void walk_fwd(const Src& S, const Taps<T>& tp, int H, int W, int x0, int y0, int y1,
                                         float mu, Emit& emit) {
  if constexpr (kInt) box_walk_int<SEG, T, kOffset, kFull, Q>(S, tp, H, W, x0, y0, y1, mu, emit);
  else box_walk<SEG, T, kOffset, kFull, Q>(S, tp, H, W, x0, y0, y1, mu, emit);
}

// Emitter that adds an item's outputs to its register accumulator (the
// input gradient, summed over boxes).
template <int SEG>
struct AccRows {
  float (&acc)[SEG][kQ];
  template <bool kFull>
  __device__ __forceinline__ void put(int s, const float* o) {
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[s][q] += o[q];
  }
};

// Backward walk over one item on the table of one upstream-gradient map G,
// with the adjoint taps of the box.  For each input pixel (y, x) =
// (y0 + s, x0 + q):
//   acc[s][q] += D(y, x), the adjoint box sum of G (the input gradient);
// and, since <G, box(I)> = <I, D> for every placement of the box, the four
// edge gradients of the original box follow from the derivatives of D with
// respect to the adjoint's edges, weighted by the map value v[s][q] = I(y, x)
// (0 outside the map).  The adjoint's edges are a' = 1 - b, b' = 1 - a,
// c' = 1 - d, d' = 1 - c, so
//   dL/da = -sum v * (G integrated over the adjoint's y extent along the
//           column just below x + b'): the y-weighted differences of the two
//           table columns at b';
//   dL/db = +sum v * (the same at a');
//   dL/dc = -sum v * (G integrated over the x extent along the row below
//           y + d'): the difference of the x-interpolated rows at d';
//   dL/dd = +sum v * (the same at c').
// These are Eq. 4's edge integrals moved to the gradient's table; the adjoint
// split of the edges puts the one-sided derivative between each edge's two
// taps.  Per pixel they are sums over the four tap rows r = c'0, c'1, d'0,
// d'1 of (column difference at a' or b', or x-interpolated row) times the
// row's y weight times v; regrouped by table row instead, each of the item's
// SEG + 1 rows of each y edge is interpolated once (rows c'0 + j and
// d'0 + j) and, with v[-1] = v[SEG] = 0 and dv = v[j-1] - v[j], the sums are
//   E0 = sum_j A_c(j) e_c(j) + A_d(j) e_d(j)  = dL/db,
//   E1 = sum_j B_c(j) e_c(j) + B_d(j) e_d(j)  = -dL/da,
//   E2 = sum_j U_c(j) dv(j)                   = dL/dd,
//   E3 = sum_j U_d(j) dv(j)                   = -dL/dc,
// with e_c(j) = wy0 v[j] + wy1 v[j-1] and e_d(j) = wy2 v[j] + wy3 v[j-1].  An
// edge's two y weights split 1 (wy0 + wy1 = -1, wy2 + wy3 = 1, up to their
// fp32 rounding), so e_c = -v[j-1] - wy0 dv and e_d = v[j-1] - wy2 dv: 9
// operations per row and column instead of 12 multiply-adds per pixel (pose
// layer backward 176 -> 174 us).
template <int SEG, bool kFull, typename Src>
__device__ __forceinline__ void adjoint_walk(const Src& S, const Taps<float>& tp, int x0, int y0, int y1,
                                                  const float (&v)[SEG][kQ], float (&acc)[SEG][kQ], float (&E)[4]) {
  const typename Src::Cols cl = S.cols(x0 + tp.ox[0], x0 + tp.ox[2]);
  const int st = S.row_step();
  const int rc = S.row_coord(y0 + tp.oy[0]), rd = S.row_coord(y0 + tp.oy[2]);
  float Uc[kQ], Ud[kQ];
#pragma unroll
  for (int j = 0; j <= SEG; ++j) {
    if (kFull || y0 + j <= y1) {
      float Uc1[kQ], Ac[kQ], Bc[kQ], Ud1[kQ], Ad[kQ], Bd[kQ];
      table_row_grad(S, rc + j * st, cl, tp, Uc1, Ac, Bc);
      table_row_grad(S, rd + j * st, cl, tp, Ud1, Ad, Bd);
#pragma unroll
      for (int q = 0; q < kQ; ++q) {
        const float vp = j > 0 ? v[j - 1][q] : 0.f;
        const float vc = j < SEG ? v[j][q] : 0.f;
        const float dv = vp - vc;
        const float ec = fmaf(-tp.wy[0], dv, -vp);
        const float ed = fmaf(-tp.wy[2], dv, vp);
        E[0] = fmaf(Ac[q], ec, fmaf(Ad[q], ed, E[0]));
        E[1] = fmaf(Bc[q], ec, fmaf(Bd[q], ed, E[1]));
        E[2] = fmaf(Uc1[q], dv, E[2]);
        E[3] = fmaf(Ud1[q], dv, E[3]);
        if (j > 0) {
          float a = acc[j - 1][q];
          a = fmaf(tp.wy[0], Uc[q], a);
          a = fmaf(tp.wy[1], Uc1[q], a);
          a = fmaf(tp.wy[2], Ud[q], a);
          acc[j - 1][q] = fmaf(tp.wy[3], Ud1[q], a);
        }
        Uc[q] = Uc1[q];
        Ud[q] = Ud1[q];
      }
    }
  }
}

// Emitter of forward outputs: the Q outputs of row y0 + s at plane offset
// off0 + s * W (elements; off0 = y0 * W + x0).
// kNT: non-temporal stores (the HBM-table forwards with outputs larger than
// the last-level cache, see kStreamOutBytes).  kPack (bf16 outputs, Q even,
// whole items): a row of the item goes out as Q / 2 packed words in one store,
// 2: W and x0 even and the output 4-byte aligned, so each word is aligned; 1:
// any W (the store is then 2-byte aligned, which global memory accesses may
// be on this target).
template <typename OutT, typename T, bool kNT = false, int Q = kQ, int kPack = 0>
struct StoreRows {
  OutT* out;
  int W, x0, off0;
  template <bool kFull>
  __device__ __forceinline__ void put(int s, const T* o) {
    if constexpr (kPack && kFull) {
      static_assert(std::is_same<OutT, uint16_t>::value && std::is_same<T, float>::value && Q % 2 == 0 && !kNT,
                    "packed rows are bf16 pairs");
      // one v_cvt_pk_bf16_f32 per pair (the rounding of convert_out)
      typedef float f32x2 __attribute__((ext_vector_type(2)));
      typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
      struct Words { uint32_t w[Q / 2]; } t;
#pragma unroll
      for (int k = 0; k < Q / 2; ++k)
        t.w[k] = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){o[2 * k], o[2 * k + 1]}, bf16x2));
      OutT* row = out + (unsigned)(off0 + s * W);
      if constexpr (kPack == 2) row = static_cast<OutT*>(__builtin_assume_aligned(row, 4));
      __builtin_memcpy(row, &t, sizeof(t));
      return;
    }
    OutT* row = out + (unsigned)(off0 + s * W);
#pragma unroll
    for (int q = 0; q < Q; ++q)
      if (kFull || x0 + q < W) {
        if constexpr (kNT) __builtin_nontemporal_store(convert_out<OutT, T>(o[q]), row + q);
        else row[q] = convert_out<OutT, T>(o[q]);
      }
  }
};

template <typename T> __device__ __forceinline__ Taps<T> typed_taps(const Taps<float>& t);
template <> __device__ __forceinline__ Taps<float> typed_taps<float>(const Taps<float>& t) { return t; }
template <> __device__ __forceinline__ Taps<int> typed_taps<int>(const Taps<float>& t) { return int_taps(t); }

// Map values of one item, 0 outside the map (they then add nothing to the
// parameter gradients).
template <int SEG>
__device__ __forceinline__ void load_item(const float* __restrict__ xs, int H, int W, int x0, int y0, bool active,
                                          float (&v)[SEG][kQ]) {
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) {
      const int yy = y0 + s, xx = x0 + q;
      v[s][q] = (active && yy < H && xx < W) ? xs[(size_t)yy * W + xx] : 0.f;
    }
}

// The same of an item that lies whole inside the map.
template <int SEG>
__device__ __forceinline__ void load_item_full(const float* __restrict__ xs, int W, int x0, int y0,
                                               float (&v)[SEG][kQ]) {
  const float* p = xs + (unsigned)(y0 * W + x0);
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) v[s][q] = p[(unsigned)(s * W) + q];
}

// Zeroes the values of an item's first `cols` columns and `rows` rows (those
// that belong to its neighbours).
template <int SEG>
__device__ __forceinline__ void keep_own(float (&v)[SEG][kQ], int cols, int rows) {
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) v[s][q] = (q >= cols && s >= rows) ? v[s][q] : 0.f;
}

// The item's origin passes through an opaque copy (an empty asm with the
// coordinates as operands): the stores then recompute their row addresses
// instead of the compiler holding load_item's 64-bit row offsets live across
// a whole kernel (seven register pairs in the 8-row backward, which spilled
// them at four waves per SIMD).
__device__ __forceinline__ void opaque_origin(int& x0, int& y0) { asm volatile("" : "+v"(x0), "+v"(y0)); }

// kFull: the item lies whole inside the map.
template <int SEG, bool kFull = false>
__device__ __forceinline__ void store_item(float* __restrict__ out, int H, int W, int x0, int y0,
                                           const float (&acc)[SEG][kQ]) {
  opaque_origin(x0, y0);
#pragma unroll
  for (int s = 0; s < SEG; ++s) {
    const int yy = y0 + s;
    if (kFull || yy < H) {
#pragma unroll
      for (int q = 0; q < kQ; ++q)
        if (kFull || x0 + q < W) out[(size_t)yy * W + x0 + q] = acc[s][q];
    }
  }
}

// The input gradient of a layer whose input x is a ReLU output, in the
// compute type of the bf16 mix before it: bf16(x > 0 ? dx : 0), round to
// nearest even.  x > 0 is the ReLU's own mask, so these are the operand bits
// that mix's backward forms.  The mask is taken from the item's input values
// once, as one bit per output (relu_mask), so they need not stay live.
template <int SEG>
__device__ __forceinline__ uint32_t relu_mask(const float (&v)[SEG][kQ]) {
  static_assert(SEG * kQ <= 32, "one bit per output");
  uint32_t m = 0;
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) m |= (v[s][q] > 0.f ? 1u : 0u) << (s * kQ + q);
  asm volatile("" : "+v"(m));  // else the compiler tests the values again at the end, and keeps them live
  return m;
}

// fp32 -> bf16 bits, round to nearest even, in integer arithmetic: the same
// bits as the conversion instruction for every finite value and infinity (a
// NaN stays a quiet NaN).  Here the instruction's form made the backward's
// register allocation grow from 144 to 224 VGPRs; this one does not.
__device__ __forceinline__ uint16_t bf16_rne_bits(float f) {
  const uint32_t b = __float_as_uint(f);
  if ((b & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((b >> 16) | 0x40u);
  return (uint16_t)((b + 0x7fffu + ((b >> 16) & 1u)) >> 16);
}

template <int SEG, bool kFull = false>
__device__ __forceinline__ void store_item_relu_bf16(uint16_t* __restrict__ out, int H, int W, int x0, int y0,
                                                     const float (&acc)[SEG][kQ], uint32_t mask) {
  opaque_origin(x0, y0);
#pragma unroll
  for (int s = 0; s < SEG; ++s) {
    const int yy = y0 + s;
    if (kFull || yy < H) {
#pragma unroll
      for (int q = 0; q < kQ; ++q)
        if (kFull || x0 + q < W)
          out[(size_t)yy * W + x0 + q] = bf16_rne_bits(((mask >> (s * kQ + q)) & 1u) ? acc[s][q] : 0.f);
    }
  }
}

// Lane move (data-parallel primitive `ctrl`), 0 where the source lane is
// disabled.
template <int kCtrl>
__device__ __forceinline__ float dpp_move(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xF, 0xF, false));
}

// The wave's sums of the four edge gradients, written to pp[0..3] (lanes 0..3
// store one each).  A transposed reduction: the pair step (lane ^ 1) leaves
// even lanes summing values 0 and 1 and odd lanes values 2 and 3, the quad
// step (lane ^ 2) one value per lane, index 2 * (lane & 1) + ((lane >> 1) &
// 1); rotations by 4 and 8 lanes inside each 16-lane row, then the row
// swaps (lane ^ 16, lane ^ 32), finish the sum in every lane.  17 vector
// operations for the four sums instead of four separate reductions (four
// lane moves and four lane reads each).  Every lane of the wave must be
// active; the order of the additions is fixed, so the sums are
// deterministic.
__device__ __forceinline__ void store_wave_partial(const float* g4, float* __restrict__ pp) {
  const int lane = threadIdx.x & 63;
  const bool odd = lane & 1, hi = lane & 2;
  float k0 = odd ? g4[2] : g4[0], k1 = odd ? g4[3] : g4[1];
  const float s0 = odd ? g4[0] : g4[2], s1 = odd ? g4[1] : g4[3];
  k0 += dpp_move<0xB1>(s0);  // quad_perm 1,0,3,2: lane ^ 1
  k1 += dpp_move<0xB1>(s1);
  float t = hi ? k1 : k0;
  const float u = hi ? k0 : k1;
  t += dpp_move<0x4E>(u);    // quad_perm 2,3,0,1: lane ^ 2
  t += dpp_move<0x124>(t);   // row_ror:4
  t += dpp_move<0x128>(t);   // row_ror:8
  auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = __uint_as_float(r16[0]) + __uint_as_float(r16[1]);  // rows 0+1 and 2+3
  auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  t = __uint_as_float(r32[0]) + __uint_as_float(r32[1]);  // halves
  if (lane < 4) pp[2 * (lane & 1) + (lane >> 1)] = t;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
inline hipError_t last_error() { return hipGetLastError(); }

// f(std::integral_constant<bool, v>) for the runtime flag v.
template <typename F>
inline void with_flag(bool v, F&& f) {
  if (v) f(std::integral_constant<bool, true>{});
  else f(std::integral_constant<bool, false>{});
}

// Output rows per item of the strided forwards.
constexpr int kSegS = 8;

// Forward launch geometry shared by both LDS kernels.
struct FwdGeom { int per_box_p, bpg, ngrp, threads; };
inline FwdGeom fwd_geom_items(int N, int C, int B, int per_box) {
  FwdGeom g;
  g.per_box_p = ((per_box + 63) / 64) * 64;
  g.bpg = 256 / g.per_box_p;
  if (g.bpg < 1) g.bpg = 1;
  if (g.bpg > B) g.bpg = B;
  // keep enough blocks in flight to fill the chip
  while (g.bpg > 1 && (long)N * C * ((B + g.bpg - 1) / g.bpg) < 2048) g.bpg = (g.bpg + 1) / 2;
  g.ngrp = (B + g.bpg - 1) / g.bpg;
  g.threads = min(g.bpg * g.per_box_p, 256);
  return g;
}
inline FwdGeom fwd_geom(int N, int C, int H, int W, int B, int seg) {
  return fwd_geom_items(N, C, B, n_chunks(W) * n_segs(H, seg));
}


// The HBM-table forwards re-read their tables through the caches; an output
// larger than the last-level cache (256 MiB) cannot stay there for the next
// call anyway, so 4-byte outputs that large are stored non-temporally and
// leave the caches to the tables (4 x 128 maps of 256x256, 8 boxes, fp32
// out: 893 -> 776 us).  Narrower outputs keep ordinary stores: 2-byte
// non-temporal stores were slower.
constexpr size_t kStreamOutBytes = (size_t)256 << 20;
inline bool stream_out(size_t elems, size_t bytes_per) { return bytes_per == 4 && elems * bytes_per > kStreamOutBytes; }

// Rows per item of the HBM-table backwards.
constexpr int kBwdGatherSeg = 8;

// Boxes per block of the box-gradient reductions.
constexpr int kReduceBoxes = 16;

}  // namespace bc
