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

// Zero row 0 and columns -PAD..0 of every row of a padded LDS table.
template <int PAD = kPad, typename T>
__device__ __forceinline__ void table_zero_edges(T* S, int H, int pitch) {
  const int tid = threadIdx.x, nt = blockDim.x;
  for (int v = tid; v < pitch; v += nt) S[v] = (T)0;
  for (int k = tid; k < H * (PAD + 1); k += nt) {
    const int u = 1 + k / (PAD + 1);
    S[u * pitch + k - (u - 1) * (PAD + 1)] = (T)0;
  }
}

// Row pass of a padded LDS table whose interior holds column prefix sums:
// lanes own rows, reading kScan elements ahead before writing, so that a
// lane's LDS reads overlap; also fills the right padding.
template <int PAD = kPad, typename T>
__device__ __forceinline__ void table_row_pass(T* S, int H, int W, int pitch) {
  constexpr int kScan = 16;
  T* R = S + PAD;
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
    for (int k = 1; k <= PAD; ++k) row[W + k] = run;
  }
}

// The row pass of a HalfRowTable: column sums of the W columns at every other
// entry, each prefix written to its two entries of the W_up = 2 W or 2 W - 1.
template <typename T>
__device__ __forceinline__ void table_row_pass_up2(T* S, int H, int W, int W_up, int pitch) {
  constexpr int kScan = 8;
  T* R = S + kPad;
  for (int u = threadIdx.x + 1; u <= H; u += blockDim.x) {
    T* row = R + u * pitch + 1;
    T run = (T)0;
    int v = 0;
    for (; v + kScan <= W; v += kScan) {
      T r[kScan];
#pragma unroll
      for (int k = 0; k < kScan; ++k) r[k] = row[2 * (v + k)];
#pragma unroll
      for (int k = 0; k < kScan; ++k) {
        run += r[k];
        row[2 * (v + k)] = run;
        row[2 * (v + k) + 1] = run;  // past the last column: padding, the same total
      }
    }
    for (; v < W; ++v) {
      run += row[2 * v];
      row[2 * v] = run;
      row[2 * v + 1] = run;
    }
#pragma unroll
    for (int k = 0; k < kPad; ++k) row[W_up + k] = run;
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
template <typename T, int kSkip = 0>
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
    int j = tid % W;
    int o = (tid / W + 1) * pitch + j + 1;
    const int step = di * pitch + dj, wrap = pitch - W;
    constexpr int kBatch1 = kSkip ? kSkip : 4;
    for (int base = 0; base < n; base += nt * kBatch1) {
      T q[kBatch1];
#pragma unroll
      for (int b = 0; b < kBatch1; ++b)
        if (!kSkip || base + b * nt < n) q[b] = __builtin_nontemporal_load(src + min(base + b * nt + tid, n - 1));
#pragma unroll
      for (int b = 0; b < kBatch1; ++b) {
        if (kSkip && base + b * nt >= n) break;
        if (tid < n - base - b * nt) R[o] = sub ? (T)((float)q[b] - mu) : q[b];
        o += step;
        j += dj;
        if (j >= W) { j -= W; o += wrap; }
      }
    }
  }
  __syncthreads();
  table_scans(S, H, W, pitch);
}

// The same table with its column sums formed in registers, for maps up to 64 *
// CPL wide: lane l owns columns l (and l + 64), wave w the RPW rows from w *
// RPW on, so a map row is one coalesced load per wave with a wave-uniform row
// offset, all RPW of them in flight.  Each lane sums down its rows, the waves
// exchange their column totals through LDS (part), and each column sum is
// written once, where staging the map and summing it in place takes four LDS
// accesses and a pass that leaves most of the block waiting.  The row pass
// (table_row_pass) stays one row per lane: scanning across lanes instead needs
// no LDS but six moves per row, and these kernels wait on their vector
// arithmetic first (box backward, 64x48 maps: 143 us staged, 146 scanned
// across lanes, 126 this way; 64x64: 128 and 98).  Row 0 and the left padding
// stay zero (table_zero_edges, once per block).
template <typename T, int RPW, int CPL, int PAD = kPad>
struct BandTable {
  T r[RPW][CPL];

  // rows [row0, row0 + RPW) of the map; rows past it repeat the last one and
  // are not written; lanes past the map read 0 (the descriptor's range check)
  __device__ __forceinline__ void load(const T* src, int H, int W, int row0) {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), (short)0, H * W * 4, 0x00020000);
    const int lane = threadIdx.x & 63;
    unsigned vo[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) vo[k] = lane + 64 * k < W ? 4u * (lane + 64 * k) : 0x40000000u;
#pragma unroll
    for (int i = 0; i < RPW; ++i)
#pragma unroll
      for (int k = 0; k < CPL; ++k)
        r[i][k] = __builtin_bit_cast(
            T, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)vo[k], min(row0 + i, H - 1) * W * 4, 2));
  }

  // column sums within the band (of the map minus mu with `sub`); the totals
  // go to part[wave]
  __device__ __forceinline__ void sum_rows(T* part, int wave, bool sub, float mu) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      if (sub) {
#pragma unroll
        for (int i = 0; i < RPW; ++i) r[i][k] = (T)((float)r[i][k] - mu);
      }
#pragma unroll
      for (int i = 1; i < RPW; ++i) r[i][k] += r[i - 1][k];
      part[(wave * CPL + k) * 64 + lane] = r[RPW - 1][k];
    }
  }

  // after a barrier: adds the bands above (and carry, the strips above, which
  // then takes this strip's total) and writes the column sums, kStep entries
  // apart
  template <int kStep = 1>
  __device__ __forceinline__ void finish(const T* part, int nw, int wave, T (&carry)[CPL], T* S, int H, int W,
                                         int pitch, int row0) {
    const int lane = threadIdx.x & 63;
    const int rows = min(RPW, H - row0);
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      T above = carry[k], total = carry[k];
      for (int h = 0; h < nw; ++h) {
        const T t = part[(h * CPL + k) * 64 + lane];
        if (h < wave) above += t;
        total += t;
      }
      carry[k] = total;
#pragma unroll
      for (int i = 0; i < RPW; ++i) r[i][k] += above;
    }
    T* row = S + PAD + 1 + lane * kStep + (row0 + 1) * pitch;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      if (lane + 64 * k < W) {
        if (rows == RPW) {
#pragma unroll
          for (int i = 0; i < RPW; ++i) row[i * pitch + 64 * k * kStep] = r[i][k];
        } else {
#pragma unroll
          for (int i = 0; i < RPW; ++i)
            if (i < rows) row[i * pitch + 64 * k * kStep] = r[i][k];
        }
      }
    }
  }
};

// Builds a map's table with BandTable, strip by strip of nw * RPW rows.  part:
// 2 * nw * 64 * CPL words of LDS.  No wave writes to S before every wave has
// reached the first strip's barrier; the table is complete after the last.
// kHalf: the table is that of the map zero-upsampled by two (HalfRowTable):
// W_up columns, each column's sums at twice its place.
template <typename T, int RPW, int CPL, bool kHalf = false, int PAD = kPad>
__device__ __forceinline__ void build_table_bands(const T* __restrict__ src, T* S, T* part, int H, int W, int pitch,
                                                  float mu, bool sub, int W_up = 0) {
  const int nw = blockDim.x >> 6, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  T carry[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) carry[k] = (T)0;
  int buf = 0;
  for (int r0 = 0; r0 < H; r0 += nw * RPW) {
    BandTable<T, RPW, CPL, PAD> band;
    const int row0 = r0 + wave * RPW;
    T* pt = part + buf * nw * 64 * CPL;
    band.load(src, H, W, row0);
    band.sum_rows(pt, wave, sub, mu);
    __syncthreads();
    band.template finish<kHalf ? 2 : 1>(pt, nw, wave, carry, S, H, W, pitch, row0);
    buf ^= 1;
  }
  __syncthreads();
  if constexpr (kHalf) table_row_pass_up2(S, H, W, W_up, pitch);
  else table_row_pass<PAD>(S, H, W, pitch);
  __syncthreads();
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

// The columns of a Q-column item as groups of Src::kRun, each with its own
// clamped run start: an LDS table's padding (PAD columns a side) covers runs
// of PAD + 1 words only, so a wider item reads its runs group by group.
template <int Q, typename Src>
struct ColGroups {
  static constexpr int G = Q < Src::kRun ? Q : Src::kRun;
  static_assert(Q % G == 0, "items are whole groups of columns");
  static constexpr int NG = Q / G;
  typename Src::Cols c[NG];
  __device__ __forceinline__ ColGroups(const Src& S, int ba, int bb) {
#pragma unroll
    for (int g = 0; g < NG; ++g) c[g] = S.cols(ba + g * G, bb + g * G);
  }
  // x-interpolated row (table_row) for all Q columns
  template <typename T>
  __device__ __forceinline__ void row(const Src& S, int coord, const Taps<T>& tp, T* U) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) table_row<G>(S, coord, c[g], tp, U + g * G);
  }
  // the G-word runs at both x edges, for all Q columns
  template <typename T>
  __device__ __forceinline__ void runs(const Src& S, int coord, T* sa, T* sb) const {
#pragma unroll
    for (int g = 0; g < NG; ++g) S.template runs<G>(coord, c[g], sa + g * G, sb + g * G);
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
  const auto rc = S.row_coord(y0 + tp.oy[0]), rd = S.row_coord(y0 + tp.oy[2]);
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
      cl.runs(S, S.row_at(rc, s), ca, cb);
      cl.runs(S, S.row_at(rd, s), da, db);
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
  const auto rc = S.row_coord(y0 + tp.oy[0]), rd = S.row_coord(y0 + tp.oy[2]);
  float Uc[kQ], Ud[kQ];
#pragma unroll
  for (int j = 0; j <= SEG; ++j) {
    if (kFull || y0 + j <= y1) {
      float Uc1[kQ], Ac[kQ], Bc[kQ], Ud1[kQ], Ad[kQ], Bd[kQ];
      table_row_grad(S, S.row_at(rc, j), cl, tp, Uc1, Ac, Bc);
      table_row_grad(S, S.row_at(rd, j), cl, tp, Ud1, Ad, Bd);
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

// Items of a map: Q columns x SEG rows each, chunks fastest.  The last chunk
// and the last segment are moved back to end at the map's edge, so that every
// item is whole: its walk has no guards, and a wave never runs a guarded walk
// beside an unguarded one (with 64 columns in 3-column chunks every wave held
// a one-column chunk and ran both).  The overlapped outputs are computed twice,
// by the same operations on the same table entries, and stored with the same
// bits.  Maps smaller than one item (W < Q or H < SEG) take the guarded
// instances (kTail).
template <int SEG, int Q>
struct ItemPos {
  int xo, yo;  // first column and row that are the item's own
  int x0, y0;  // first column and row it covers
  __device__ __forceinline__ ItemPos(int it, int nch, int H, int W, bool tail) {
    const int seg = it / nch, ch = it - seg * nch;
    xo = ch * Q;
    yo = seg * SEG;
    x0 = tail ? xo : min(xo, W - Q);
    y0 = tail ? yo : min(yo, H - SEG);
  }
};

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

// Most threads of a forward block.
constexpr int kFwdThreads = 512;

// Columns per lane of the register-built tables (BandTable) of each compiled
// pitch: 55 and 71 serve maps up to 64 wide, 103 up to 96.
constexpr int band_cols(int pitch) { return pitch <= 71 ? 1 : 2; }
// LDS of a table and of the band totals its builder exchanges.
// (The 6-column forward items' tables are 6 wider, see kFwdPad.)
inline size_t table_lds_bytes(int rows, int W, int pitch_class, int threads) {
  if (pitch_class == 0) return (size_t)(rows + 1) * lds_pitch(W) * 4;
  return ((size_t)(rows + 1) * pitch_class + 2 * threads * band_cols(pitch_class)) * 4;
}

// f(std::integral_constant<int, pitch>) for a compiled pitch (0: run-time pitch).
template <typename F>
inline void with_pitch(int pitch, F&& f) {
  switch (pitch) {
    case 55: f(std::integral_constant<int, 55>{}); return;
    case 71: f(std::integral_constant<int, 71>{}); return;
    case 103: f(std::integral_constant<int, 103>{}); return;
    default: f(std::integral_constant<int, 0>{});
  }
}

// Forward launch geometry shared by both LDS kernels.
struct FwdGeom { int per_box_p, bpg, ngrp, threads; };
// Blocks of up to max_threads, each with a map's table of its own, so a block
// takes as many of the map's boxes as fit its threads while every CU still
// gets a block.
inline FwdGeom fwd_geom_items(int N, int C, int B, int per_box, int max_threads) {
  FwdGeom g;
  g.per_box_p = ((per_box + 63) / 64) * 64;
  g.bpg = max_threads / g.per_box_p;
  if (g.bpg < 1) g.bpg = 1;
  if (g.bpg > B) g.bpg = B;
  while (g.bpg > 1 && (long)N * C * ((B + g.bpg - 1) / g.bpg) < 256) g.bpg = (g.bpg + 1) / 2;
  g.ngrp = (B + g.bpg - 1) / g.bpg;
  // as many boxes in each (5 as 3 + 2, not 4 + 1): a block of few idles, its
  // table no cheaper (6 x 245 maps of 54x96, 5 boxes: 71 us, even 63)
  g.bpg = (B + g.ngrp - 1) / g.ngrp;
  g.threads = min(g.bpg * g.per_box_p, max_threads);
  return g;
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
