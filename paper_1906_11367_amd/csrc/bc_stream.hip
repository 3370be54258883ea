// Streaming box kernels: the summed-area table is never stored.  A group of
// lanes walks one box down the map, output row by output row, keeping the two
// table rows each y edge needs as running column prefix sums (two cursors);
// each step forms one row from them and scans it once across the group.
//
// Why this is the same computation (Section 3.1, Eq. 2-3).  With the
// exclusive table S(u, v) = sum_{i<u, j<v} I(i, j), the column prefix
// P(u, j) = sum_{i<u} I(i, j) and the row prefix of a row vector R,
// (scan R)(v) = sum_{j<v} R(j), the table row is S(u, .) = scan P(u, .).  A
// box's bilinear corner samples at output row y are
//   sum_r wy[r] * sum_k wx[k] * S(u_r, x + ox[k]),   u_r = y + oy[r] (clamped),
// and since the row scan is linear, sum_r wy[r] S(u_r, .) = scan Y with
//   Y = sum_r wy[r] P(u_r, .).
// The rows u_r come in pairs (f, f + 1) at each y edge, P(f + 1) = P(f) +
// I(f), and the two weights of a pair sum to -1 (upper edge) and +1 (lower
// edge), so
//   Y = P(y + fd) - P(y + fc) - beta_c * I(y + fc) + beta_d * I(y + fd)
// (beta the edges' fractions).  Per output row each cursor adds one map row,
// Y takes three operations per column, one scan gives scan Y, and the x
// taps are read from it exactly as from a table row.  Clamping a table
// index to [0, H] x [0, W] is zero padding; here a cursor outside the map
// adds nothing, and the scanned row is padded with 0 on the left and its
// last value on the right.
//
// Backward (the adjoint box on the upstream gradient G, as the table
// kernels do):
//   input gradient  sum_b of the adjoint box sums of G_b;
//   edge gradients  dL/da = -sum v * DB, dL/db = sum v * DA, where DA, DB
//                   are the differences of scan Y across the adjoint's two x
//                   edges (the y-weighted column differences) and v the input;
//                   dL/dc = -sum_j G(y + fd, j) * T(j), dL/dd =
//                   sum_j G(y + fc, j) * T(j), with T(j) = sum_k wx[k] *
//                   V(j + 1 - ox[k]) and V(t) = sum_{x >= t} v(y, x): the
//                   x-interpolated row of the table of the single row G(y + f)
//                   weighted by v, moved onto the input row (sum_x v(x) sum_k
//                   wx[k] sum_{j < x+ox[k]} G(j) = sum_j G(j) T(j)).  The
//                   weights of a box sum to 0, so V may be replaced by minus
//                   the prefix sums of the input row, one forward scan.
// Lane layout: a group of LG lanes holds one box's row, CPL consecutive
// columns per lane (LG * CPL >= W); LG = 16 puts four boxes in a wave (one
// per DPP row, scans by row shifts), LG = 64 one box per wave.
#include "bc_common.hpp"
#include "bc_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace bc {
namespace {

// Sum over the lanes of a group, in every lane of the group.
template <int LG>
__device__ __forceinline__ float group_sum(float v) {
  v = row16_sum(v);
  if constexpr (LG == 64) {
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
  }
  return v;
}

}  // namespace

// Padding of a group's scanned row in LDS, on each side: a run of CPL + 1
// consecutive entries whose start is clamped to [-pad, W] then reads exactly
// the clamped entries.
template <int CPL> constexpr int stream_pad() { return CPL + 1; }
// With an even CPL, lanes address a row CPL words apart, which puts lanes 32
// / CPL apart on one LDS bank; one skip word every 32 words (index i at
// i + i / 32) spreads them over all banks.  Odd CPL needs none.
template <int CPL> constexpr bool stream_skew() { return CPL % 2 == 0; }
template <int LG, int CPL> constexpr int stream_row_words() {
  constexpr int n = 2 * stream_pad<CPL>() + LG * CPL + 1;
  return stream_skew<CPL>() ? n + n / 32 + 1 : n;
}
// LDS index of row entry v (v in [-pad, LG * CPL + pad]).
template <int CPL>
__device__ __forceinline__ int stream_at(int v) {
  const int i = v + stream_pad<CPL>();
  return stream_skew<CPL>() ? i + (i >> 5) : i;
}
// LDS index of element j of a group's input-gradient slot (j in [0, LG*CPL)).
template <int CPL>
__device__ __forceinline__ int slot_at(int j) { return stream_skew<CPL>() ? j + (j >> 5) : j; }
template <int LG, int CPL> constexpr int slot_words() { return stream_skew<CPL>() ? LG * CPL + LG * CPL / 32 : LG * CPL; }

// Rows of a step are loaded this many steps ahead, so that its loads are in
// flight while the steps before it compute: in a ring of registers with the
// loop unrolled over it, or (kRing, below) in a queue copied forward.
constexpr int kPrefetch = 2;
// Forward: three (us two and three ahead: 2 x 64 maps of 300x130, 4 boxes 123 and
// 119; 1 x 32 of 256x256, 8 boxes 112 and 108; 4 x 128 of those 322 and 322), but
// two where three leave one block per CU that does not fill it (kAhead).
constexpr int kFwdPrefetch = 3;

// The lane's CPL columns of a map row: byte offsets within a row (columns
// outside the map clamped onto its last column, so every load is in bounds)
// and which of them lie in the map.  A row is then CPL loads from one uniform
// base plus a per-lane 32-bit offset.
template <int CPL>
struct LaneCols {
  unsigned off[CPL];
  bool in[CPL];
  __device__ __forceinline__ LaneCols(int x0, int W) {
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      in[k] = x0 + k < W;
      off[k] = 4u * (unsigned)min(x0 + k, W - 1);
    }
  }
  // row `row` of the map at byte offset `mapoff` from base (rows outside
  // [0, H) and columns outside the map read as 0).  The load is always made
  // (from a valid address) and its bits masked, so no branch surrounds it.
  // kVec: every lane's CPL columns lie in the map (W == LG * CPL) and rows
  // are 16-byte aligned, so a row is one 16-byte load per lane (CPL = 4).
  template <bool kVec, typename T>
  __device__ __forceinline__ void load(const T* base, unsigned mapoff, int row, int H, int W, bool live,
                                       T* r) const {
    const bool ok = live && row >= 0 && row < H;
    const unsigned ro = ok ? mapoff + 4u * (unsigned)(row * W) : 0u;
    const char* b = reinterpret_cast<const char*>(base);
    if constexpr (kVec && CPL == 4) {
      typedef int i4 __attribute__((ext_vector_type(4)));
      const i4 t = *reinterpret_cast<const i4*>(b + (ro + off[0]));
      const int m = ok ? -1 : 0;
      r[0] = __builtin_bit_cast(T, t.x & m);
      r[1] = __builtin_bit_cast(T, t.y & m);
      r[2] = __builtin_bit_cast(T, t.z & m);
      r[3] = __builtin_bit_cast(T, t.w & m);
    } else {
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const int t = *reinterpret_cast<const int*>(b + (ro + off[k]));
        const int m = (ok && in[k]) ? -1 : 0;
        r[k] = __builtin_bit_cast(T, t & m);
      }
    }
  }
};

// The same for groups of a whole wave: the box, and with it the row, is
// wave-uniform, so a row is one scalar offset into the map's buffer
// descriptor (rows outside the map: an offset past its end, which reads 0),
// and columns outside the map are lane offsets past its end.  Row checks and
// addresses then cost scalar instructions; they were a third of the vector
// instructions of these kernels, which wait on those first.
template <int CPL>
struct WaveRows {
  __amdgpu_buffer_rsrc_t rs;
  unsigned off[CPL];
  int H, row_bytes;
  __device__ __forceinline__ WaveRows(const void* map, int x0, int H_, int W) : H(H_), row_bytes(4 * W) {
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(map), (short)0, H_ * W * 4, 0x00020000);
#pragma unroll
    for (int k = 0; k < CPL; ++k) off[k] = x0 + k < W ? 4u * (unsigned)(x0 + k) : 0x40000000u;
  }
  __device__ __forceinline__ bool inside(int row) const { return row >= 0 && row < H; }
  template <bool kVec, typename T>
  __device__ __forceinline__ void load(int row, T* r) const {
    const unsigned ro = inside(row) ? (unsigned)(row * row_bytes) : 0x40000000u;
    if constexpr (kVec && CPL == 4) {
      const auto t = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off[0] + ro), 0, 0);
      const unsigned w[4] = {t[0], t[1], t[2], t[3]};
#pragma unroll
      for (int k = 0; k < 4; ++k) r[k] = __builtin_bit_cast(T, w[k]);
    } else {
#pragma unroll
      for (int k = 0; k < CPL; ++k)
        r[k] = __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off[k] + ro), 0, 0));
    }
  }
};

// A value that is the same in every lane of a group: a scalar when the group
// is the wave.
template <int LG> __device__ __forceinline__ int group_uniform(int v) {
  return LG == 64 ? __builtin_amdgcn_readfirstlane(v) : v;
}

// ---------------------------------------------------------------------------
// Backward.  One block of NG groups per map (n, c); group g walks box b = g.
// dx: each group leaves its adjoint sums in LDS slots; every R rows the
// block adds the NG slots of each element in a fixed order and writes dx
// (two slot sets alternate, so one barrier per R rows orders every write
// before its reads and every read before the slot's next write).  kInt:
// boxes with integer corners (input gradient only, x not read).  kRelu: dx
// written as bf16(x > 0 ? dx : 0).  partials: [n][C*B][4] edge gradients
// (one row per image).
// ---------------------------------------------------------------------------
template <int LG, int CPL, int NG, bool kInt, bool kRelu, bool kVec, bool kRing>
__global__ __launch_bounds__(LG * NG) void k_box_bwd_stream(const float* __restrict__ x, const int* __restrict__ taps,
                                                            const float* __restrict__ gy, void* __restrict__ gx,
                                                            float* __restrict__ partials, int C, int H, int W, int B,
                                                            int R) {
  static_assert(!(kInt && kRelu), "the ReLU mask needs x");
  constexpr int PAD = stream_pad<CPL>();
  constexpr int RW = stream_row_words<LG, CPL>();
  constexpr int PF = kPrefetch;
  constexpr int LC = LG * CPL;            // columns a group covers
  constexpr int SW = slot_words<LG, CPL>();
  extern __shared__ __align__(16) float smem[];
  float* SY = smem;                       // [NG][RW]: scan Y of each group's box
  float* SV = SY + NG * RW;               // [NG][RW]: prefix sums of the input row
  float* DX = SV + NG * RW;               // [2][R][NG][SW]: adjoint sums, added over groups
  const int map = blockIdx.x, n = map / C, c = map - n * C;
  const int g = group_uniform<LG>(threadIdx.x / LG), p = threadIdx.x % LG;
  const int b = g;
  const bool live = b < B;
  const int x0 = p * CPL;
  const size_t plane = (size_t)H * W;
  const float* xs = x + (size_t)map * plane;
  const float* gbase = gy + (size_t)map * B * plane;
  const unsigned gmap = live ? 4u * (unsigned)(b * plane) : 0u;
  const LaneCols<CPL> cols(x0, W);
  const WaveRows<CPL> xrows(xs, x0, H, W), grows(gbase + (size_t)(live ? b : 0) * plane, x0, H, W);
  auto load_x = [&](int row, float (&r)[CPL]) {
    if constexpr (LG == 64) xrows.template load<kVec>(row, r);
    else cols.template load<kVec>(xs, 0u, row, H, W, true, r);
  };
  auto load_g = [&](int row, float (&r)[CPL]) {
    if constexpr (LG == 64) grows.template load<kVec>(live ? row : -1, r);
    else cols.template load<kVec>(gbase, gmap, row, H, W, live, r);
  };
  float* sy = SY + g * RW;                // sy[stream_at(v)] = scan Y (v), v in [-PAD, LC + PAD]
  float* sv = SV + g * RW;
  // adjoint record of the box (each group its own; vector loads)
  const Taps<float> tp = load_taps(taps + (size_t)C * B * 16 + (size_t)(c * B + (live ? b : 0)) * 16, W, H);
  const int fa = tp.ox[0], fb = tp.ox[2], fc = tp.oy[0], fd = tp.oy[2];
  const float aa = -tp.wx[1], ab = tp.wx[3], bc_ = -tp.wy[1], bd = tp.wy[3];
  // LDS indices of the lane's tap runs (scan Y at the adjoint's x edges, the
  // input row's sums at the mirrored taps) and of the entries it writes
  int ia[CPL + 1], ib[CPL + 1], ja[CPL + 1], jb[CPL + 1], iw[CPL];
  {
    const int ra0 = clampi(x0 + fa, -PAD, W), rb0 = clampi(x0 + fb, -PAD, W);
    const int va0 = clampi(x0 - fa, -PAD, W), vb0 = clampi(x0 - fb, -PAD, W);
#pragma unroll
    for (int k = 0; k <= CPL; ++k) {
      ia[k] = stream_at<CPL>(ra0 + k);
      ib[k] = stream_at<CPL>(rb0 + k);
      ja[k] = stream_at<CPL>(va0 + k);
      jb[k] = stream_at<CPL>(vb0 + k);
    }
#pragma unroll
    for (int k = 0; k < CPL; ++k) iw[k] = stream_at<CPL>(x0 + k + 1);
  }
  // constant parts of the LDS rows: both are 0 left of column 0
  for (int t = p; t <= PAD; t += LG) {
    sy[stream_at<CPL>(-PAD + t)] = 0.f;
    sv[stream_at<CPL>(-PAD + t)] = 0.f;
  }
  // cursors: P(clamp(y + fc)) and P(clamp(y + fd)) at the lane's columns
  float pc[CPL], pd[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) { pc[k] = 0.f; pd[k] = 0.f; }
  {
    const int upto = live ? min(max(fd, 0), H) : 0;
    for (int u0 = 0; u0 < upto; u0 += PF) {
      float r[PF][CPL];
#pragma unroll
      for (int i = 0; i < PF; ++i) load_g(u0 + i < upto ? u0 + i : -1, r[i]);
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        const bool inc = u0 + i < fc;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
          pd[k] += r[i][k];
          if (inc) pc[k] += r[i][k];
        }
      }
    }
  }
  float ca = 0.f, cb = 0.f, gcs = 0.f, gds = 0.f;
  // rows of step y: the input row v, gc_ = G(y + fc), gd_ = G(y + fd).  kRing:
  // a ring of PF + 1 steps with the loop unrolled over it; else a queue whose
  // rows are copied forward (up to 24 moves a step, but one copy of the step).
  constexpr int RS = kRing ? PF + 1 : PF;
  float qv[RS][CPL], qc[RS][CPL], qd[RS][CPL];
  auto issue = [&](int y, float (&v)[CPL], float (&gc_)[CPL], float (&gd_)[CPL]) {
    const bool in = y < H;
    if constexpr (!kInt) load_x(in ? y : -1, v);
    load_g(in ? y + fc : -1, gc_);
    load_g(in ? y + fd : -1, gd_);
  };
  int bi = 0, ri = 0;   // slot set and row of the current batch
  // one output row
  auto step = [&](int y, const float* v, const float* gc_, const float* gd_) {
    // Y and its scan (inclusive within the lane, then across the group)
    float s[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      float yv = pd[k] - pc[k];
      if constexpr (!kInt) yv = fmaf(bd, gd_[k], fmaf(-bc_, gc_[k], yv));
      s[k] = k ? s[k - 1] + yv : yv;
      pc[k] += gc_[k];
      pd[k] += gd_[k];
    }
    const float tot = s[CPL - 1];
    const float off = group_excl<LG>(tot);
#pragma unroll
    for (int k = 0; k < CPL; ++k) sy[iw[k]] = s[k] + off;
    if (p == LG - 1) {
#pragma unroll
      for (int t = 1; t <= PAD; ++t) sy[stream_at<CPL>(LC + t)] = s[CPL - 1] + off;
    }
    // prefix sums of the input row (the same in every group)
    if constexpr (!kInt) {
      float pfx[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) pfx[k] = k ? pfx[k - 1] + v[k] : v[k];
      const float voff = group_excl<LG>(pfx[CPL - 1]);
#pragma unroll
      for (int k = 0; k < CPL; ++k) sv[iw[k]] = pfx[k] + voff;
      if (p == LG - 1) {
#pragma unroll
        for (int t = 1; t <= PAD; ++t) sv[stream_at<CPL>(LC + t)] = pfx[CPL - 1] + voff;
      }
    }
    __builtin_amdgcn_wave_barrier();
    // the adjoint box sums of the lane's outputs and the edge terms
    float sa[CPL + 1], sb[CPL + 1];
#pragma unroll
    for (int k = 0; k <= CPL; ++k) { sa[k] = sy[ia[k]]; sb[k] = sy[ib[k]]; }
    float* dxs = DX + ((bi * R + ri) * NG + g) * SW;
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      float d;
      if constexpr (kInt) {
        d = sb[k] - sa[k];
      } else {
        const float da = sa[k + 1] - sa[k], db = sb[k + 1] - sb[k];
        d = fmaf(ab, db, fmaf(-aa, da, sb[k] - sa[k]));
        ca = fmaf(v[k], da, ca);
        cb = fmaf(v[k], db, cb);
      }
      dxs[slot_at<CPL>(x0 + k)] = live ? d : 0.f;
    }
    if constexpr (!kInt) {
      float A[CPL + 1], Bv[CPL + 1];
#pragma unroll
      for (int k = 0; k <= CPL; ++k) { A[k] = sv[ja[k]]; Bv[k] = sv[jb[k]]; }
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const float t = fmaf(ab, Bv[k + 1] - Bv[k], fmaf(-aa, A[k + 1] - A[k], A[k + 1] - Bv[k + 1]));
        gcs = fmaf(gc_[k], t, gcs);
        gds = fmaf(gd_[k], t, gds);
      }
    }
    __builtin_amdgcn_wave_barrier();
    // every R rows (and after the last): the slots of the batch, added over
    // the groups in a fixed order
    if (++ri == R || y == H - 1) {
      __syncthreads();
      const float* slots = DX + bi * R * NG * SW;
      for (int r = 0; r < ri; ++r) {
        const int yy = y + 1 - ri + r;
        for (int j = threadIdx.x; j < W; j += LG * NG) {
          float acc = 0.f;
#pragma unroll
          for (int h = 0; h < NG; ++h) acc += slots[(r * NG + h) * SW + slot_at<CPL>(j)];
          const size_t o = (size_t)map * plane + (size_t)yy * W + j;
          if constexpr (kRelu) {
            static_cast<uint16_t*>(gx)[o] = f32_to_bf16_rne(xs[(size_t)yy * W + j] > 0.f ? acc : 0.f);
          } else if (gx != nullptr) {
            static_cast<float*>(gx)[o] = acc;
          }
        }
      }
      ri = 0;
      bi ^= 1;
    }
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) issue(i, qv[i], qc[i], qd[i]);
  if constexpr (kRing) {
    int y = 0;
    for (; y + RS <= H; y += RS) {
#pragma unroll
      for (int i = 0; i < RS; ++i) {
        issue(y + i + PF, qv[(i + PF) % RS], qc[(i + PF) % RS], qd[(i + PF) % RS]);
        step(y + i, qv[i], qc[i], qd[i]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int i = 0; i < PF; ++i)
      if (y + i < H) step(y + i, qv[i], qc[i], qd[i]);
  } else {
    for (int y = 0; y < H; ++y) {
      float v[CPL], gc_[CPL], gd_[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) { v[k] = qv[0][k]; gc_[k] = qc[0][k]; gd_[k] = qd[0][k]; }
#pragma unroll
      for (int i = 0; i + 1 < PF; ++i)
#pragma unroll
        for (int k = 0; k < CPL; ++k) { qv[i][k] = qv[i + 1][k]; qc[i][k] = qc[i + 1][k]; qd[i][k] = qd[i + 1][k]; }
      issue(y + PF, qv[PF - 1], qc[PF - 1], qd[PF - 1]);
      step(y, v, gc_, gd_);
    }
  }
  if constexpr (!kInt) {
    // (dL/da, dL/db, dL/dc, dL/dd) of the box, one partial per image
    ca = group_sum<LG>(ca);
    cb = group_sum<LG>(cb);
    gcs = group_sum<LG>(gcs);
    gds = group_sum<LG>(gds);
    if (live && p == 0) {
      float* pp = partials + ((size_t)n * C * B + (size_t)c * B + b) * 4;
      pp[0] = -cb;
      pp[1] = ca;
      pp[2] = -gds;
      pp[3] = gcs;
    }
  }
}

// ---------------------------------------------------------------------------
// Forward.  One block of NG groups per map (n, c); group g walks box b = g
// over the map's rows and writes that box's output row by row (no table, no
// exchange between groups).  T = int: integer maps (the sum of Eq. 1 over the
// floored box, exact).  kInt: boxes with integer corners (four table
// samples, no interpolation).  kOffset: the map's mean mu is subtracted
// before the cursors add its rows and mu times the clipped box area is added
// back (the same combination applied to the clamped coordinates).  kNT:
// non-temporal output stores (outputs larger than the last-level cache).
// kAhead: steps a row is loaded ahead.  kRing: the rows in a ring, else in a
// queue (see the backward): non-temporal stores word by word write their lines
// to memory in parts, the more the further the waves run apart, and the queue
// holds them closer together (4 x 128 maps of 256 x 128, 8 boxes: 269 us in a
// ring, 235 in a queue).
// ---------------------------------------------------------------------------
template <typename T, typename OutT, int LG, int CPL, int NG, bool kOffset, bool kInt, bool kNT, bool kVec, int kAhead>
__global__ __launch_bounds__(LG * NG) void k_box_fwd_stream(const T* __restrict__ x, const int* __restrict__ taps,
                                                            OutT* __restrict__ y, int C, int H, int W, int B) {
  constexpr bool kRing = !kNT || kVec;
  constexpr bool kPlain = kInt || std::is_same<T, int>::value;   // corner weights (-1, 0, 1, 0)
  constexpr int PAD = stream_pad<CPL>();
  constexpr int RW = stream_row_words<LG, CPL>();
  constexpr int PF = kAhead;
  constexpr int LC = LG * CPL;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* SY = reinterpret_cast<T*>(smem_raw);
  __shared__ float red[(LG * NG + 63) / 64];
  const int map = blockIdx.x, c = map % C;
  const int g = group_uniform<LG>(threadIdx.x / LG), p = threadIdx.x % LG;
  const int b = g;
  const bool live = b < B;
  const int x0 = p * CPL;
  const size_t plane = (size_t)H * W;
  const T* xs = x + (size_t)map * plane;
  const LaneCols<CPL> cols(x0, W);
  const WaveRows<CPL> rows(xs, x0, H, W);
  T* sy = SY + g * RW;                    // sy[stream_at(v)] = scan Y (v)
  float mu = 0.f;
  if constexpr (kOffset) {
    float sum = 0.f;
    for (size_t i = threadIdx.x; i < plane; i += LG * NG) sum += (float)xs[i];
    sum = wave_sum(sum);
    constexpr int nw = (LG * NG + 63) / 64;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
    __syncthreads();
    float tot = 0.f;
#pragma unroll
    for (int w = 0; w < nw; ++w) tot += red[w];
    mu = tot / (float)plane;
  }
  const Taps<float> tp = load_taps(taps + (size_t)(c * B + (live ? b : 0)) * 16, W, H);
  const int fa = tp.ox[0], fb = tp.ox[2], fc = tp.oy[0], fd = tp.oy[2];
  const float aa = -tp.wx[1], ab = tp.wx[3], bc_ = -tp.wy[1], bd = tp.wy[3];
  int ia[CPL + 1], ib[CPL + 1], iw[CPL];
  {
    const int ra0 = clampi(x0 + fa, -PAD, W), rb0 = clampi(x0 + fb, -PAD, W);
#pragma unroll
    for (int k = 0; k <= CPL; ++k) {
      ia[k] = stream_at<CPL>(ra0 + k);
      ib[k] = stream_at<CPL>(rb0 + k);
    }
#pragma unroll
    for (int k = 0; k < CPL; ++k) iw[k] = stream_at<CPL>(x0 + k + 1);
  }
  for (int t = p; t <= PAD; t += LG) sy[stream_at<CPL>(-PAD + t)] = (T)0;
  T pc[CPL], pd[CPL];
#pragma unroll
  for (int k = 0; k < CPL; ++k) { pc[k] = (T)0; pd[k] = (T)0; }
  // map row `row` at the lane's columns, 0 outside, and (kOffset, where it is
  // used) minus mu
  auto load_row = [&](int row, T (&r)[CPL]) {
    if constexpr (LG == 64) rows.template load<kVec>(live ? row : -1, r);
    else cols.template load<kVec>(xs, 0u, row, H, W, live, r);
  };
  float mul[CPL];   // mu at the lane's columns, 0 outside the map
#pragma unroll
  for (int k = 0; k < CPL; ++k) mul[k] = kVec || cols.in[k] ? mu : 0.f;
  auto minus_mu = [&](int row, T (&r)[CPL]) {
    if constexpr (kOffset) {
      const bool ok = live && row >= 0 && row < H;
#pragma unroll
      for (int k = 0; k < CPL; ++k) r[k] = (T)((float)r[k] - (ok ? (kVec ? mu : mul[k]) : 0.f));
    }
  };
  {
    const int upto = live ? min(max(fd, 0), H) : 0;
    for (int u0 = 0; u0 < upto; u0 += PF) {
      T r[PF][CPL];
#pragma unroll
      for (int i = 0; i < PF; ++i) load_row(u0 + i < upto ? u0 + i : -1, r[i]);
#pragma unroll
      for (int i = 0; i < PF; ++i) {
        minus_mu(u0 + i < upto ? u0 + i : -1, r[i]);
        const bool inc = u0 + i < fc;
#pragma unroll
        for (int k = 0; k < CPL; ++k) {
          pd[k] += r[i][k];
          if (inc) pc[k] += r[i][k];
        }
      }
    }
  }
  // clipped extent of the box along x at the lane's outputs (kOffset)
  float ex[CPL];
  if constexpr (kOffset) {
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      const int xa = x0 + k + fa, xb = x0 + k + fb;
      const float wa = (float)(clampi(xa + 1, 0, W) - clampi(xa, 0, W));
      const float wb = (float)(clampi(xb + 1, 0, W) - clampi(xb, 0, W));
      ex[k] = (float)(clampi(xb, 0, W) - clampi(xa, 0, W)) + (kPlain ? 0.f : ab * wb - aa * wa);
    }
  }
  OutT* out = y + ((size_t)map * B + (live ? b : 0)) * plane;
  auto step = [&](int yy, T (&gc_)[CPL], T (&gd_)[CPL]) {
    minus_mu(yy + fc, gc_);
    minus_mu(yy + fd, gd_);
    T s[CPL];
#pragma unroll
    for (int k = 0; k < CPL; ++k) {
      T yv = pd[k] - pc[k];
      if constexpr (!kPlain) yv = fmaf(bd, gd_[k], fmaf(-bc_, gc_[k], yv));
      s[k] = k ? s[k - 1] + yv : yv;
      pc[k] += gc_[k];
      pd[k] += gd_[k];
    }
    const T tot = s[CPL - 1];
    const T off = group_excl<LG>(tot);
#pragma unroll
    for (int k = 0; k < CPL; ++k) sy[iw[k]] = s[k] + off;
    if (p == LG - 1) {
#pragma unroll
      for (int t = 1; t <= PAD; ++t) sy[stream_at<CPL>(LC + t)] = s[CPL - 1] + off;
    }
    __builtin_amdgcn_wave_barrier();
    T sa[CPL + 1], sb[CPL + 1];
#pragma unroll
    for (int k = 0; k <= CPL; ++k) { sa[k] = sy[ia[k]]; sb[k] = sy[ib[k]]; }
    float ey = 0.f;
    if constexpr (kOffset) {
      const int yc = yy + fc, yd = yy + fd;
      const float wc = (float)(clampi(yc + 1, 0, H) - clampi(yc, 0, H));
      const float wd = (float)(clampi(yd + 1, 0, H) - clampi(yd, 0, H));
      ey = mu * ((float)(clampi(yd, 0, H) - clampi(yc, 0, H)) + (kPlain ? 0.f : bd * wd - bc_ * wc));
    }
    if (live) {
      OutT* row = out + (size_t)yy * W;
      OutT ov[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        T o;
        if constexpr (kPlain) o = sb[k] - sa[k];
        else o = fmaf(ab, sb[k + 1] - sb[k], fmaf(-aa, sa[k + 1] - sa[k], sb[k] - sa[k]));
        if constexpr (kOffset) o = add_offset(o, ex[k], ey);
        if constexpr (std::is_same<OutT, uint16_t>::value) ov[k] = f32_to_bf16_rne((float)o);
        else ov[k] = (OutT)o;
      }
      if constexpr (kVec && CPL == 4 && sizeof(OutT) == 4) {
        typedef OutT v4 __attribute__((ext_vector_type(4)));
        const v4 q = {ov[0], ov[1], ov[2], ov[3]};
        v4* dst = reinterpret_cast<v4*>(row + x0);
        if constexpr (kNT) __builtin_nontemporal_store(q, dst);
        else *dst = q;
      } else if constexpr (kVec && CPL == 4) {   // 2-byte outputs: one 8-byte store
        const uint2 q = make_uint2((uint32_t)ov[0] | ((uint32_t)ov[1] << 16), (uint32_t)ov[2] | ((uint32_t)ov[3] << 16));
        *reinterpret_cast<uint2*>(row + x0) = q;
      } else {
#pragma unroll
        for (int k = 0; k < CPL; ++k)
          if (cols.in[k]) {
            if constexpr (kNT) __builtin_nontemporal_store(ov[k], row + x0 + k);
            else row[x0 + k] = ov[k];
          }
      }
    }
    __builtin_amdgcn_wave_barrier();
  };
  // main loop, the rows of step yy loaded PF steps ahead
  constexpr int RS = kRing ? PF + 1 : PF;
  T qc[RS][CPL], qd[RS][CPL];
  auto issue = [&](int yn, T (&gc_)[CPL], T (&gd_)[CPL]) {
    load_row(yn < H ? yn + fc : -1, gc_);
    load_row(yn < H ? yn + fd : -1, gd_);
  };
#pragma unroll
  for (int i = 0; i < PF; ++i) issue(i, qc[i], qd[i]);
  if constexpr (kRing) {
    int yy = 0;
    for (; yy + RS <= H; yy += RS) {
#pragma unroll
      for (int i = 0; i < RS; ++i) {
        issue(yy + i + PF, qc[(i + PF) % RS], qd[(i + PF) % RS]);
        step(yy + i, qc[i], qd[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < PF; ++i)
      if (yy + i < H) step(yy + i, qc[i], qd[i]);
  } else {
    for (int yy = 0; yy < H; ++yy) {
      T gc_[CPL], gd_[CPL];
#pragma unroll
      for (int k = 0; k < CPL; ++k) { gc_[k] = qc[0][k]; gd_[k] = qd[0][k]; }
#pragma unroll
      for (int i = 0; i + 1 < PF; ++i)
#pragma unroll
        for (int k = 0; k < CPL; ++k) { qc[i][k] = qc[i + 1][k]; qd[i][k] = qd[i + 1][k]; }
      issue(yy + PF, qc[PF - 1], qd[PF - 1]);
      step(yy, gc_, gd_);
    }
  }
}

// ---------------------------------------------------------------------------
// Launchers.  Geometry: LG = 16 for maps up to 64 wide (four boxes per wave),
// LG = 64 up to 256 wide (a box per wave); CPL = ceil(W / LG); NG = 4 or 8
// groups (boxes) per block, so B <= 8.  The backward adds the groups' input
// gradients every R <= 8 rows, as many as kSlotBytes hold.
// ---------------------------------------------------------------------------
// LDS for one slot set: the groups' input gradients of R rows, added after a
// block barrier (256x256 maps, 8 boxes: a barrier every row 492 us, every
// other row 473, every 4 rows 579, which leave one block per CU).
constexpr size_t kSlotBytes = 20 << 10;
struct StreamGeom { int lg, cpl, ng, R; };

static bool stream_geom(int H, int W, int B, StreamGeom& g) {
  if (W <= 64) {
    g.lg = 16;
    g.cpl = W <= 16 ? 1 : W <= 32 ? 2 : W <= 48 ? 3 : 4;
  } else if (W <= 256) {
    g.lg = 64;
    g.cpl = W <= 128 ? 2 : W <= 192 ? 3 : 4;
  } else {
    return false;
  }
  if (B > 8) return false;
  g.ng = B <= 4 ? 4 : 8;
  // per-lane 32-bit byte offsets into a block's gradient maps
  if ((size_t)g.ng * H * W * 4 >= ((size_t)1 << 31)) return false;
  const size_t slot_set = (size_t)g.ng * (g.lg * g.cpl + g.lg * g.cpl / 32) * 4;
  // small blocks of many boxes: every row, for more blocks per CU (16 x 128 maps
  // of 420 x 64, 8 boxes: 753 us, every 8 rows 938)
  if (g.lg == 16 && g.ng == 8 && g.cpl >= 3) g.R = 1;
  else g.R = (int)std::max<size_t>(1, std::min<size_t>(8, kSlotBytes / slot_set));
  return true;
}

bool box_stream_supported(int H, int W, int B) {
  StreamGeom g;
  return stream_geom(H, W, B, g);
}

// Vector row accesses: every lane's columns inside the map and 16-byte
// aligned rows (W == LG * CPL, CPL = 4, base pointers 16-byte aligned).
static bool stream_vec(int W, int lg, int cpl) { return cpl == 4 && W == lg * cpl; }

// Layouts that store such outputs non-temporally word by word (those that store
// whole rows always do): 65 to 128 columns.  The others' partial lines cost more
// than the cache they leave free (4 x 128 maps of 256 x 160, 8 boxes: 514 us,
// with ordinary stores 364; 16 x 128 of 800 x 30, 4 boxes: 790, 504).
constexpr bool stream_nt_words(int lg, int cpl) { return lg == 64 && cpl == 2; }

template <int LG, int CPL, int NG>
static void bwd_stream_t(const float* x, const int* taps, const float* gy, void* gx, float* partials, int N, int C,
                         int H, int W, int B, bool rounded, bool relu_bf16, int R, hipStream_t s) {
  constexpr int RW = stream_row_words<LG, CPL>();
  const size_t shm = ((size_t)2 * NG * RW + (size_t)2 * R * NG * slot_words<LG, CPL>()) * sizeof(float);
  const dim3 grid(N * C), block(LG * NG);
  // Rows in a ring or a queue.  With all gradients the ring's unrolled loop takes
  // 187 VGPRs for 4 columns and 148 for 3: one block of 512 threads per CU.  4 x
  // 128 maps, ring and queue: 256 x 256, 8 boxes 565 and 473 us; 256 x 160, 8
  // boxes 519 and 465; 256 x 130, 4 boxes (blocks of 256) 227 and 253.  16 x 128
  // maps of 400 x 46, 6 boxes 722 and 630.  Calls whose blocks are all resident
  // with the ring as well keep it: 3 x 44 maps of 132 x 136, 8 boxes, masked, 131
  // and 163; 5 x 80 of 400 x 46 (blocks of 128, six a CU) 305 and 361.
  auto go = [&](auto ki, auto kr, auto kv) {
    auto launch = [&](auto kring) {
      hipLaunchKernelGGL((k_box_bwd_stream<LG, CPL, NG, decltype(ki)::value, decltype(kr)::value, decltype(kv)::value,
                                           decltype(kring)::value>),
                         grid, block, shm, s, x, taps, gy, gx, partials, C, H, W, B, R);
    };
    constexpr bool kInt = decltype(ki)::value;
    if constexpr (CPL == 3 && NG == 8 && !kInt) {
      if ((long)N * C <= (LG == 16 ? 6 * 256 : 256)) launch(std::true_type{});
      else launch(std::false_type{});
    } else {
      launch(std::integral_constant<bool, CPL <= 3 || kInt>{});
    }
  };
  auto with_vec = [&](auto ki, auto kr) {
    if constexpr (CPL == 4) {
      if (stream_vec(W, LG, CPL)) {
        go(ki, kr, std::true_type{});
        return;
      }
    }
    go(ki, kr, std::false_type{});
  };
  if (rounded) with_vec(std::true_type{}, std::false_type{});
  else if (relu_bf16) with_vec(std::false_type{}, std::true_type{});
  else with_vec(std::false_type{}, std::false_type{});
}

hipError_t launch_box_bwd_stream(const float* x, const int* taps, const float* gy, void* gx, float* partials, int N,
                                 int C, int H, int W, int B, bool rounded, bool relu_bf16, hipStream_t s) {
  StreamGeom g;
  if (!stream_geom(H, W, B, g) || (rounded && relu_bf16)) return hipErrorInvalidValue;
#define BC_BWD_STREAM(LG, CPL, NG)                                                                            \
  if (g.lg == LG && g.cpl == CPL && g.ng == NG) {                                                           \
    bwd_stream_t<LG, CPL, NG>(x, taps, gy, gx, partials, N, C, H, W, B, rounded, relu_bf16, g.R, s);       \
    return hipGetLastError();                                                                               \
  }
  BC_BWD_STREAM(16, 1, 4) BC_BWD_STREAM(16, 2, 4) BC_BWD_STREAM(16, 3, 4) BC_BWD_STREAM(16, 4, 4)
  BC_BWD_STREAM(16, 1, 8) BC_BWD_STREAM(16, 2, 8) BC_BWD_STREAM(16, 3, 8) BC_BWD_STREAM(16, 4, 8)
  BC_BWD_STREAM(64, 2, 4) BC_BWD_STREAM(64, 3, 4) BC_BWD_STREAM(64, 4, 4)
  BC_BWD_STREAM(64, 2, 8) BC_BWD_STREAM(64, 3, 8) BC_BWD_STREAM(64, 4, 8)
#undef BC_BWD_STREAM
  return hipErrorInvalidValue;
}

template <typename T, typename OutT, int LG, int CPL, int NG, bool kOffset>
static void fwd_stream_t(const void* x, const int* taps, void* y, int N, int C, int H, int W, int B, bool rounded,
                         bool nt, hipStream_t s) {
  const size_t shm = (size_t)NG * stream_row_words<LG, CPL>() * sizeof(T);
  auto launch = [&](auto ki, auto kn, auto kv, auto ka) {
    hipLaunchKernelGGL((k_box_fwd_stream<T, OutT, LG, CPL, NG, kOffset, decltype(ki)::value, decltype(kn)::value,
                                         decltype(kv)::value, decltype(ka)::value>),
                       dim3(N * C), dim3(LG * NG), shm, s, (const T*)x, taps, (OutT*)y, C, H, W, B);
  };
  using Two = std::integral_constant<int, 2>;
  auto go = [&](auto ki, auto kn, auto kv) {
    // mean removed, 4 columns: 140 VGPRs, one block of 512 threads per CU; with 5
    // of its 8 boxes at work that does not fill it (4 x 128 maps of 256x256: 304
    // us three ahead, 267 two; 8 boxes 354 and 368)
    if constexpr (kOffset && LG == 64 && CPL == 4 && NG == 8 && decltype(kv)::value) {
      if (B == 5) {
        launch(ki, kn, kv, Two{});
        return;
      }
    }
    if constexpr (decltype(kn)::value && !decltype(kv)::value) launch(ki, kn, kv, Two{});
    else launch(ki, kn, kv, std::integral_constant<int, kFwdPrefetch>{});
  };
  auto with_vec = [&](auto ki) {
    const std::true_type yes;
    const std::false_type no;
    constexpr bool kF32 = std::is_same<OutT, float>::value;
    if constexpr (CPL == 4) {
      if (stream_vec(W, LG, CPL)) {
        if constexpr (kF32) {
          if (nt) {
            go(ki, yes, yes);
            return;
          }
        }
        go(ki, no, yes);
        return;
      }
    }
    if constexpr (kF32 && stream_nt_words(LG, CPL)) {
      if (nt) {
        go(ki, yes, no);
        return;
      }
    }
    go(ki, no, no);
  };
  if (rounded) with_vec(std::true_type{});
  else with_vec(std::false_type{});
}

template <int LG, int CPL, int NG>
static void fwd_stream_dispatch(const void* x, bool is_int, const int* taps, void* y, int out_kind, int N, int C,
                                int H, int W, int B, bool offset, bool rounded, bool nt, hipStream_t s) {
  if (is_int) fwd_stream_t<int, int, LG, CPL, NG, false>(x, taps, y, N, C, H, W, B, rounded, false, s);
  else if (out_kind == 2) {
    if (offset) fwd_stream_t<float, uint16_t, LG, CPL, NG, true>(x, taps, y, N, C, H, W, B, rounded, false, s);
    else fwd_stream_t<float, uint16_t, LG, CPL, NG, false>(x, taps, y, N, C, H, W, B, rounded, false, s);
  } else {
    if (offset) fwd_stream_t<float, float, LG, CPL, NG, true>(x, taps, y, N, C, H, W, B, rounded, nt, s);
    else fwd_stream_t<float, float, LG, CPL, NG, false>(x, taps, y, N, C, H, W, B, rounded, nt, s);
  }
}

hipError_t launch_box_fwd_stream(const void* x, bool is_int, const int* taps, void* y, int out_kind, int N, int C,
                                 int H, int W, int B, bool offset, bool rounded, hipStream_t s) {
  StreamGeom g;
  if (!stream_geom(H, W, B, g)) return hipErrorInvalidValue;
  // fp32 outputs larger than the last-level cache
  const bool nt = out_kind == 1 && (size_t)N * C * B * H * W * 4 > ((size_t)256 << 20);
#define BC_FWD_STREAM(LG, CPL, NG)                                                                                \
  if (g.lg == LG && g.cpl == CPL && g.ng == NG) {                                                               \
    fwd_stream_dispatch<LG, CPL, NG>(x, is_int, taps, y, out_kind, N, C, H, W, B, offset, rounded, nt, s);     \
    return hipGetLastError();                                                                                   \
  }
  BC_FWD_STREAM(16, 1, 4) BC_FWD_STREAM(16, 2, 4) BC_FWD_STREAM(16, 3, 4) BC_FWD_STREAM(16, 4, 4)
  BC_FWD_STREAM(16, 1, 8) BC_FWD_STREAM(16, 2, 8) BC_FWD_STREAM(16, 3, 8) BC_FWD_STREAM(16, 4, 8)
  BC_FWD_STREAM(64, 2, 4) BC_FWD_STREAM(64, 3, 4) BC_FWD_STREAM(64, 4, 4)
  BC_FWD_STREAM(64, 2, 8) BC_FWD_STREAM(64, 3, 8) BC_FWD_STREAM(64, 4, 8)
#undef BC_FWD_STREAM
  return hipErrorInvalidValue;
}

}  // namespace bc
