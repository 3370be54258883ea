// Box filter kernels on tables built in LDS: forward (plain and strided) and
// backward (input and box-parameter gradients).  gfx950, wave64.
#include "bc_box.hpp"

#include <algorithm>

namespace bc {

// Padding of the forward's tables of compiled pitch: a 6-column item then
// reads each of its runs as 7 words from one clamped address instead of two
// runs of 4.
constexpr int kFwdPad = 6;

// Forward on a map's table in LDS, for the groups g0 .. g0+ng-1 of bpw boxes
// of channel c.  Items of one box are (row segment, column chunk), chunk
// fastest so that adjacent lanes write adjacent columns; a group's items are
// padded to a multiple of 64 (per_grp) so that a wave works on one group.  One
// box (bpw = 1): the wave reads its taps through scalar loads.  kLanes: maps of
// at most 32 items, whose waves would be half empty, take as many boxes as fit
// 64 lanes, each lane with its own box's taps (13 x 225 maps of 8x74, 8 boxes: 50
// us with a box per wave, 25 so).
template <typename T, typename OutT, int SEG, bool kOffset, bool kInt, int Q, int kPack, bool kTail, bool kHere,
          bool kLanes, typename Src>
__device__ __forceinline__ void fwd_boxes(const Src& tab, const int* __restrict__ taps,
                                          const float* __restrict__ boxes,
                                          OutT* __restrict__ y, int map, int c, int g0, int ng, int H, int W,
                                          int B, int bpw, int per_grp, float mu) {
  const int nch = (W + Q - 1) / Q, nseg = (H + SEG - 1) / SEG, per_box = nch * nseg;
  for (int it = threadIdx.x; it < ng * per_grp; it += blockDim.x) {
    const int gl = __builtin_amdgcn_readfirstlane(it / per_grp);
    int r = it - gl * per_grp, b = (g0 + gl) * bpw;
    if constexpr (kLanes) {
      const int bl = r / per_box;
      r -= bl * per_box;
      b += bl;
      if (bl >= bpw || b >= B) continue;
    } else {
      if (r >= per_box) continue;
    }
    const ItemPos<SEG, Q> ip(r, nch, H, W, kTail);
    const Taps<T> tp = typed_taps<T>(kHere ? make_taps_here<!kLanes>(boxes + (size_t)(c * B + b) * 4, false, kInt, W, H)
                                           : load_taps(taps + (size_t)(c * B + b) * 16, W, H));
    OutT* out = y + ((size_t)map * B + b) * H * W;
    StoreRows<OutT, T, false, Q, kPack> em{out, W, ip.x0, ip.y0 * W + ip.x0};
    walk_fwd<SEG, T, kOffset, !kTail, kInt, Q>(tab, tp, H, W, ip.x0, ip.y0, min(ip.y0 + SEG, H), mu, em);
  }
}

// Forward, table in LDS: one block per (map, bpg groups of bpw boxes).  The
// block builds the map's table once and evaluates every box of its groups.
// kPitch > 0: the table's row pitch compiled in (as in the LDS backward).  Q:
// columns per item; kPack: how rows are stored (StoreRows).
// kHere: the taps are computed from boxes (make_taps_here), else read.
template <typename T, typename OutT, int SEG, bool kOffset, bool kInt, int kPitch, int Q, int kPack, bool kTail,
          bool kHere, bool kLanes>
__global__ __launch_bounds__(kFwdThreads) void k_box_fwd_lds(const T* __restrict__ x, const int* __restrict__ taps,
                                                     const float* __restrict__ boxes,
                                                     OutT* __restrict__ y, int C, int H, int W, int B, int bpw,
                                                     int bpg, int per_grp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* S = reinterpret_cast<T*>(smem_raw);
  __shared__ float red[16];
  constexpr int PAD = kPitch > 0 ? kFwdPad : kPad;
  const int pitch = kPitch > 0 ? kPitch + 2 * (PAD - kPad) : lds_pitch_dev(W);
  const int groups = (B + bpw - 1) / bpw, ngrp = (groups + bpg - 1) / bpg;
  const int map = blockIdx.x / ngrp, grp = blockIdx.x - map * ngrp;
  const T* src = x + (size_t)map * H * W;
  float mu = 0.f;
  if (kOffset) mu = block_mean(reinterpret_cast<const float*>(src), H * W, red);
  if constexpr (kPitch > 0) {
    table_zero_edges<PAD>(S, H, pitch);
    build_table_bands<T, 16, band_cols(kPitch), false, PAD>(src, S, S + (H + 1) * pitch, H, W, pitch, mu, kOffset);
  } else {
    // Words ahead where rows have no alignment.  Eight take 82 VGPRs instead of
    // 53, which the small tables (kTail) pay for in waves (12 x 212 maps of 14x2, 5
    // boxes 38 us with eight, 29 with two); the others have at most three blocks
    // on a CU by their LDS (2 x 314 of 171x82, 3 boxes 87 with eight, 107 with two).
    build_table_lds<T, kTail ? 2 : 8>(src, S, H, W, pitch, mu, kOffset);
  }
  const int g0 = grp * bpg;
  fwd_boxes<T, OutT, SEG, kOffset, kInt, Q, kPack, kTail, kHere, kLanes>(LdsTable<T, PAD>{S, pitch, W, H}, taps, boxes,
                                                                         y, map, map % C, g0, min(bpg, groups - g0), H,
                                                                         W, B, bpw, per_grp, mu);
}

// Strided forward (stride s > 1) on a map's table in LDS, boxes b0 .. b0+nb-1
// of channel c: items are (output column, segment of kSegS output rows),
// column fastest; a box's items are padded to per_box_p (a multiple of 64)
// so each wave serves one box.
template <typename T, typename OutT, bool kOffset, bool kInt>
__device__ __forceinline__ void fwd_boxes_strided(const LdsTable<T>& tab, const int* __restrict__ taps,
                                                  OutT* __restrict__ y, int map, int c, int b0, int nb, int H, int W,
                                                  int B, int s, int Ho, int Wo, int per_box_p, float mu) {
  const int per_box = Wo * ((Ho + kSegS - 1) / kSegS);
  for (int it = threadIdx.x; it < nb * per_box_p; it += blockDim.x) {
    const int bl = __builtin_amdgcn_readfirstlane(it / per_box_p);
    const int r = it - bl * per_box_p;
    if (r >= per_box) continue;
    const int seg = r / Wo, j = r - seg * Wo;
    const int b = b0 + bl;
    const Taps<T> tp = typed_taps<T>(load_taps(taps + (size_t)(c * B + b) * 16, W, H));
    const int i0 = seg * kSegS;
    StoreCol<OutT, T> em{y + ((size_t)map * B + b) * Ho * Wo, Wo, i0 * Wo + j};
    box_walk_strided<kSegS, T, kOffset, kInt>(tab, tp, H, W, s * j, i0, min(i0 + kSegS, Ho), s, mu, em);
  }
}

template <typename T, typename OutT, bool kOffset, bool kInt, int kPitch>
__global__ __launch_bounds__(256) void k_box_fwd_lds_strided(const T* __restrict__ x, const int* __restrict__ taps,
                                                             OutT* __restrict__ y, int C, int H, int W, int B, int s,
                                                             int Ho, int Wo, int bpg, int per_box_p) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* S = reinterpret_cast<T*>(smem_raw);
  __shared__ float red[16];
  const int pitch = kPitch > 0 ? kPitch : lds_pitch_dev(W);
  const int ngrp = (B + bpg - 1) / bpg;
  const int map = blockIdx.x / ngrp, grp = blockIdx.x - map * ngrp;
  const T* src = x + (size_t)map * H * W;
  float mu = 0.f;
  if (kOffset) mu = block_mean(reinterpret_cast<const float*>(src), H * W, red);
  if constexpr (kPitch > 0) {
    table_zero_edges(S, H, pitch);
    build_table_bands<T, 16, band_cols(kPitch)>(src, S, S + (H + 1) * pitch, H, W, pitch, mu, kOffset);
  } else {
    build_table_lds(src, S, H, W, pitch, mu, kOffset);
  }
  const int b0 = grp * bpg;
  fwd_boxes_strided<T, OutT, kOffset, kInt>(LdsTable<T>{S, pitch, W, H}, taps, y, map, map % C, b0,
                                            min(bpg, B - b0), H, W, B, s, Ho, Wo, per_box_p, mu);
}

// Backward, table in LDS: one block per map (n, c); items (row segment,
// chunk), one per thread, whose map values stay in registers.  For each box
// b the table of grad_y[n][c*B+b] is built in LDS and the adjoint walk adds
// the input gradient (in registers, summed over b) and the edge gradients;
// each wave writes its edge-gradient sums to
// partials[(n * nw + wave) * C*B + c*B + b][4].  kInt (boxes with integer
// corners): the adjoint four-corner sums only, no edge gradients.  kUp
// (stride s > 1): grad_y is [maps][Ho][Wo] and is tabulated zero-upsampled,
// which makes every gradient that of the strided layer.  kRelu: gx is bf16,
// store_item_relu_bf16 (not with kInt, which does not read x).
// Four waves per SIMD: bounded to 128 VGPRs (from 144, three waves) the
// 8-row items fit without spilling once the final stores recompute their
// addresses (below); pose-layer backward 172.5 -> 151.5 us, results
// bit-identical.  The 4-row items take 92.
// kPitch > 0: the table's row pitch as a compile-time constant, so that every
// row offset of the scans and the walk is an immediate of its LDS access
// instead of a per-element address add.
// Items end at the map's edges (ItemPos): every lane runs the one unguarded
// walk.  Values an item shares with its neighbour enter the edge sums as 0
// there, so each is counted once; its input gradient is written twice with the
// same bits.
// kTail: maps smaller than an item, every row and column guarded.
// kNext (4-row items, the map one strip of its block's bands): the next
// gradient map is loaded while this one is walked.  Such calls have few blocks
// per CU to hide that load behind; the 8-row items have no registers for it,
// and more blocks.
// kUp: 0 stride 1; 1 the table of the whole zero-upsampled map; 2 (stride 2)
// its HalfRowTable.
// kHere: the taps are computed from boxes (make_taps_here), else read.
template <int SEG, bool kInt, int kUp, int kMaxT, bool kRelu, int kPitch, bool kTail, bool kNext, bool kHere>
__global__ __launch_bounds__(kMaxT) __attribute__((amdgpu_waves_per_eu(4, 8))) void k_box_bwd_lds(
    const float* __restrict__ x, const int* __restrict__ taps, const float* __restrict__ boxes,
    const float* __restrict__ gy, void* __restrict__ gx, float* __restrict__ partials, int C, int H, int W, int B, int s,
    int Ho, int Wo) {
  static_assert(!(kInt && kRelu), "the ReLU mask needs x");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int pitch = kPitch > 0 ? kPitch : lds_pitch_dev(W);
  float* SG = reinterpret_cast<float*>(smem_raw);
  const int map = blockIdx.x, n = map / C, c = map - n * C;
  const int nw = blockDim.x >> 6, wave = threadIdx.x >> 6;
  const int nch = (W + kQ - 1) / kQ, nseg = (H + SEG - 1) / SEG;
  const bool active = (int)threadIdx.x < nch * nseg;
  const ItemPos<SEG, kQ> ip(active || kTail ? threadIdx.x : 0, nch, H, W, kTail);
  const int x0 = ip.x0, y0 = ip.y0, y1 = min(y0 + SEG, H);
  const size_t plane = (size_t)H * W;
  const size_t gplane = kUp ? (size_t)Ho * Wo : plane;
  const float* g0 = gy + (size_t)map * B * gplane;
  float v[SEG][kQ], acc[SEG][kQ];
  uint32_t rmask = 0;
  if constexpr (!kInt) {
    if constexpr (kTail) load_item<SEG>(x + (size_t)map * plane, H, W, x0, y0, active, v);
    else load_item_full<SEG>(x + (size_t)map * plane, W, x0, y0, v);
    if constexpr (kRelu) rmask = relu_mask<SEG>(v);
    if constexpr (!kTail) keep_own<SEG>(v, ip.xo - x0, ip.yo - y0);
  }
#pragma unroll
  for (int s = 0; s < SEG; ++s)
#pragma unroll
    for (int q = 0; q < kQ; ++q) acc[s][q] = 0.f;
  using Table = typename std::conditional<kUp == 2, HalfRowTable, LdsTable<float>>::type;
  const Table tg{SG, pitch, W, kUp == 2 ? Ho : H};
  const int* adj = taps + (size_t)C * B * 16;
  constexpr bool kBands = kPitch > 0 && kUp != 1;
  static_assert(kBands || kUp != 2, "half-row tables are built from bands");
  const int trows = kUp == 2 ? Ho : H;  // rows of the table (below row 0)
  // rows per band: what the walk's registers leave (two columns a lane and
  // 8-row items: 16 rows spill 8 registers, 72x80 maps 57 us against 52)
  constexpr int kRows = SEG == 8 ? (band_cols(kPitch) == 1 ? 32 : 8) : 16;
  BandTable<float, kRows, band_cols(kPitch)> band;
  float* part = SG + (trows + 1) * pitch;
  const int uwave = __builtin_amdgcn_readfirstlane(wave);
  if constexpr (kBands) table_zero_edges(SG, trows, pitch);
  if constexpr (kNext) band.load(g0, H, W, uwave * kRows);
  for (int b = 0; b < B; ++b) {
    if constexpr (!kBands) __syncthreads();
    if constexpr (kUp == 1) {
      build_table_lds_up(g0 + b * gplane, SG, H, W, pitch, s, Ho, Wo);
    } else if constexpr (kNext) {
      float carry[band_cols(kPitch)] = {};
      band.sum_rows(part, uwave, false, 0.f);
      __syncthreads();
      band.finish(part, nw, uwave, carry, SG, H, W, pitch, uwave * kRows);
      __syncthreads();
      table_row_pass(SG, H, W, pitch);
      __syncthreads();
      if (b + 1 < B) band.load(g0 + (b + 1) * plane, H, W, uwave * kRows);
    } else if constexpr (kUp == 2) {
      build_table_bands<float, SEG == 8 && band_cols(kPitch) == 2 ? 8 : 16, band_cols(kPitch), true>(
          g0 + b * gplane, SG, part, Ho, Wo, pitch, 0.f, false, W);
    } else if constexpr (kBands) {
      build_table_bands<float, kRows, band_cols(kPitch)>(g0 + b * plane, SG, part, H, W, pitch, 0.f, false);
    } else {
      build_table_lds(g0 + b * plane, SG, H, W, pitch, 0.f, false);
    }
    const Taps<float> tp = kHere ? make_taps_here(boxes + (size_t)(c * B + b) * 4, true, kInt, W, H)
                                 : load_taps(adj + (size_t)(c * B + b) * 16, W, H);
    if constexpr (kInt) {  // integer corners: input gradient only
      AccRows<SEG> em{acc};
      if (active) box_walk_int<SEG, float, false, !kTail>(tg, tp, H, W, x0, y0, y1, 0.f, em);
      continue;
    }
    float E[4] = {0.f, 0.f, 0.f, 0.f};
    if (active) adjoint_walk<SEG, !kTail>(tg, tp, x0, y0, y1, v, acc, E);
    float g4[4] = {-E[1], E[0], -E[3], E[2]};   // dL/da, dL/db, dL/dc, dL/dd
    store_wave_partial(g4, partials + (((size_t)n * nw + wave) * C * B + (size_t)c * B + b) * 4);
  }
  if (active && gx != nullptr) {
    if constexpr (kRelu) store_item_relu_bf16<SEG, !kTail>(static_cast<uint16_t*>(gx) + (size_t)map * plane, H, W, x0, y0, acc, rmask);
    else store_item<SEG, !kTail>(static_cast<float*>(gx) + (size_t)map * plane, H, W, x0, y0, acc);
  }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// Calls of at most this many filtered maps compute their taps in the kernel
// instead of in a launch of box_prep before it (about 4 us; the arithmetic is
// 0.3 us a wave, which larger calls would pay many times over).
constexpr long kTapsHereBoxes = 4096;

// Rows per item of the forward: a box's items fill whole waves, and each item
// reads one row more than it writes (and its start costs about two rows), so
// the segment length with the least waves x (rows + 3) is taken; 8 rows on
// 64x48 maps (64 items, one wave), 13 on 64x64 (55 items; 8 rows would need
// 88 items in two waves).
static int fwd_seg(int H, int nch) {
  int best = 8;
  long cost = 0;
  for (int seg : {8, 10, 13}) {
    if (H < seg) continue;
    const long c = (long)((nch * n_segs(H, seg) + 63) / 64) * (seg + 3);
    if (cost == 0 || c < cost) { cost = c; best = seg; }
  }
  return best;
}

// Whether the forward's items are 3 columns of 16 rows instead of 6 columns of
// seg.  Six columns halve the table reads but leave fp32 and int32 rows as a
// 16- and an 8-byte store per lane, each of which writes parts of its lines;
// three go out as 12 bytes a lane, whole lines together.  Calls of many maps
// are bound by those stores (32 x 256 maps of 64x48, 4 boxes: 127 us with six
// columns, 104 with three) unless the narrow items cost more waves x rows x
// columns, a tenth or above (15 x 84 maps of 54x64: 114 against 96, 25 us become
// 30; 72x80: 171 and 132, 161 us become 238 with the mean); calls of few maps run on latency and keep the wide items, and tables
// of run-time pitch gain nothing (21 x 133 maps of 109x96: 64 us either way).
constexpr int kTallSeg = 16;
static bool fwd_tall_items(long boxes, int H, int W, int seg) {
  if (boxes <= kTapsHereBoxes || H < kTallSeg) return false;
  const long wide = (long)(((W + 5) / 6 * n_segs(H, seg) + 63) / 64) * (seg + 3) * 6;
  const long tall = (long)((n_chunks(W) * n_segs(H, kTallSeg) + 63) / 64) * (kTallSeg + 3) * kQ;
  return 10 * tall <= 11 * wide;
}

template <typename T, typename OutT, bool kOffset>
static void fwd_lds_t(const void* x, const int* taps, const float* boxes, void* y, int N, int C, int H, int W, int B, bool rounded,
                      int stride, hipStream_t s) {
  const int pc = lds_pitch_class(H, W);
  if (stride == 1) {
    constexpr int Q = 6;
    if (W < Q || H < 8) {  // smaller than one item
      constexpr int SEG = 16;
      const FwdGeom g = fwd_geom_items(N, C, B, n_chunks(W) * n_segs(H, SEG), 256);
      const size_t shm0 = (size_t)(H + 1) * lds_pitch(W) * sizeof(T);
      with_flag(rounded, [&](auto ki) {
        hipLaunchKernelGGL((k_box_fwd_lds<T, OutT, SEG, kOffset, decltype(ki)::value, 0, kQ, 0, true, false, false>),
                           dim3(N * C * g.ngrp), dim3(g.threads), shm0, s, (const T*)x, taps, boxes, (OutT*)y, C, H, W, B,
                           1, g.bpg, g.per_box_p);
      });
      return;
    }
    constexpr bool kOneSeg = kOffset || std::is_same<T, int>::value;
    const int nch = (W + Q - 1) / Q, seg = pc && !kOneSeg ? fwd_seg(H, nch) : 8;
    const bool lanes = pc > 0 && seg == 8 && nch * n_segs(H, seg) <= 32 && B > 1;
    const bool tall = sizeof(OutT) == 4 && pc > 0 && !lanes && fwd_tall_items((long)N * C * B, H, W, seg);
    const int per_box = tall ? n_chunks(W) * n_segs(H, kTallSeg) : nch * n_segs(H, seg);
    const int bpw = lanes ? std::min(64 / per_box, B) : 1;
    const FwdGeom g = fwd_geom_items(N, C, (B + bpw - 1) / bpw, bpw * per_box, kFwdThreads);
    const size_t shm = table_lds_bytes(H, W, pc, g.threads) + (pc ? (size_t)(H + 1) * 2 * (kFwdPad - kPad) * 4 : 0);
    auto go = [&](auto ki, auto kseg, auto kp, auto kpack) {
      auto launch = [&](auto kh, auto kl) {
        hipLaunchKernelGGL((k_box_fwd_lds<T, OutT, decltype(kseg)::value, kOffset, decltype(ki)::value,
                                          decltype(kp)::value, Q, decltype(kpack)::value, false, decltype(kh)::value,
                                          decltype(kl)::value>),
                           dim3(N * C * g.ngrp), dim3(g.threads), shm, s, (const T*)x, taps, boxes, (OutT*)y, C, H, W,
                           B, bpw, g.bpg, g.per_box_p);
      };
      auto with_lanes = [&](auto kh) {
        if constexpr (decltype(kp)::value > 0 && decltype(kseg)::value == 8) {
          if (lanes) {
            launch(kh, std::true_type{});
            return;
          }
        }
        launch(kh, std::false_type{});
      };
      if constexpr (decltype(kp)::value > 0) {
        if (boxes) {
          with_lanes(std::true_type{});
          return;
        }
      }
      with_lanes(std::false_type{});
    };
    if constexpr (sizeof(OutT) == 4) {
      if (tall) {
        with_flag(rounded, [&](auto ki) {
          with_pitch(pc, [&](auto kp) {
            if constexpr (decltype(kp)::value > 0)
              hipLaunchKernelGGL((k_box_fwd_lds<T, OutT, kTallSeg, kOffset, decltype(ki)::value, decltype(kp)::value, kQ,
                                                0, false, false, false>),
                                 dim3(N * C * g.ngrp), dim3(g.threads), shm, s, (const T*)x, taps, boxes, (OutT*)y, C, H,
                                 W, B, 1, g.bpg, g.per_box_p);
          });
        });
        return;
      }
    }
    with_flag(rounded, [&](auto ki) {
      auto packed = [&](auto kseg, auto kp) {
        // bf16 rows of an even width go out as aligned packed words
        if constexpr (std::is_same<OutT, uint16_t>::value) {
          if ((W & 1) == 0) go(ki, kseg, kp, std::integral_constant<int, 2>{});
          else go(ki, kseg, kp, std::integral_constant<int, 1>{});
        } else {
          go(ki, kseg, kp, std::integral_constant<int, 0>{});
        }
      };
      with_pitch(pc, [&](auto kp) {
        if constexpr (kOneSeg || decltype(kp)::value == 0) packed(std::integral_constant<int, 8>{}, kp);
        else if (seg == 13) packed(std::integral_constant<int, 13>{}, kp);
        else if (seg == 10) packed(std::integral_constant<int, 10>{}, kp);
        else packed(std::integral_constant<int, 8>{}, kp);
      });
    });
    return;
  }
  const int Ho = (H + stride - 1) / stride, Wo = (W + stride - 1) / stride;
  const FwdGeom g = fwd_geom_items(N, C, B, Wo * ((Ho + kSegS - 1) / kSegS), 256);
  const size_t shm = table_lds_bytes(H, W, pc, g.threads);
  with_flag(rounded, [&](auto ki) {
    auto go = [&](auto kp) {
      hipLaunchKernelGGL((k_box_fwd_lds_strided<T, OutT, kOffset, decltype(ki)::value, decltype(kp)::value>),
                         dim3(N * C * g.ngrp), dim3(g.threads), shm, s, (const T*)x, taps, (OutT*)y, C, H, W, B, stride,
                         Ho, Wo, g.bpg, g.per_box_p);
    };
    with_pitch(pc, go);
  });
}

bool box_fwd_lds_computes_taps(int N, int C, int H, int W, int B, int stride) {
  return stride == 1 && W >= 6 && H >= 8 && lds_pitch_class(H, W) > 0 && (long)N * C * B <= kTapsHereBoxes;
}

hipError_t launch_box_fwd_lds(const void* x, bool is_int, const int* taps, const float* boxes, void* y, int out_kind, int N, int C,
                              int H, int W, int B, bool offset, bool rounded, int stride, hipStream_t s) {
  if (is_int) {
    fwd_lds_t<int, int, false>(x, taps, boxes, y, N, C, H, W, B, rounded, stride, s);
  } else if (out_kind == 2) {
    if (offset) fwd_lds_t<float, uint16_t, true>(x, taps, boxes, y, N, C, H, W, B, rounded, stride, s);
    else fwd_lds_t<float, uint16_t, false>(x, taps, boxes, y, N, C, H, W, B, rounded, stride, s);
  } else {
    if (offset) fwd_lds_t<float, float, true>(x, taps, boxes, y, N, C, H, W, B, rounded, stride, s);
    else fwd_lds_t<float, float, false>(x, taps, boxes, y, N, C, H, W, B, rounded, stride, s);
  }
  return last_error();
}

template <int SEG, int kMaxT>
static void bwd_lds_t(const float* x, const int* taps, const float* boxes, const float* gy, void* gx, float* partials, int N, int C,
                      int H, int W, int B, bool rounded, bool relu_bf16, int stride, hipStream_t s) {
  const int items = n_chunks(W) * n_segs(H, SEG);
  const int threads = ((items + 63) / 64) * 64;
  const int Ho = (H + stride - 1) / stride, Wo = (W + stride - 1) / stride;
  const bool tail = W < kQ || H < SEG;
  int pc = tail ? 0 : lds_pitch_class(H, W);
  // Tables from registers load a row per wave: narrow maps of more rows than
  // their waves' bands leave most lanes idle strip after strip, and are staged
  // instead (at run-time pitch).  2046 maps of 98x12, 4 boxes: 54 us from
  // registers, 37 staged; 3114 of 50x24, 8 boxes 89 and 71; 4096 of 100x30, 4
  // boxes 121 and 147, of 32x12 (one strip) 31 and 36.  Calls of few
  // maps (4-row items, more waves a map) keep the registers: 128 maps of 64x16,
  // 8 boxes 28 and 35.
  if (SEG == 8 && stride == 1 && W <= 24 && H > threads / 64 * 32) pc = 0;
  if (stride > 2) pc = 0;  // the whole upsampled map is tabulated at run-time pitch
  const bool half = stride == 2 && pc > 0;
  const size_t shm = table_lds_bytes(half ? Ho : H, W, pc, threads);
  using std::integral_constant;
  auto go = [&](auto ki, auto kr) {
    auto launch = [&](auto ku, auto kp, auto kt, auto kn, auto kh) {
      hipLaunchKernelGGL((k_box_bwd_lds<SEG, decltype(ki)::value, decltype(ku)::value, kMaxT, decltype(kr)::value,
                                        decltype(kp)::value, decltype(kt)::value, decltype(kn)::value,
                                        decltype(kh)::value>),
                         dim3(N * C), dim3(threads), shm, s, x, taps, boxes, gy, gx, partials, C, H, W, B, stride, Ho, Wo);
    };
    const integral_constant<int, 0> c0;
    if (stride > 1 && !half) {
      if (tail) launch(integral_constant<int, 1>{}, c0, std::true_type{}, std::false_type{}, std::false_type{});
      else launch(integral_constant<int, 1>{}, c0, std::false_type{}, std::false_type{}, std::false_type{});
    } else if (tail) {
      launch(c0, c0, std::true_type{}, std::false_type{}, std::false_type{});
    } else {
      with_pitch(pc, [&](auto kp) {
        if constexpr (decltype(kp)::value > 0) {
          if (half) {
            launch(integral_constant<int, 2>{}, kp, std::false_type{}, std::false_type{}, std::false_type{});
            return;
          }
        }
        if constexpr (SEG == 4 && decltype(kp)::value > 0) {
          if (H <= threads / 64 * 16) {
            if (boxes) launch(c0, kp, std::false_type{}, std::true_type{}, std::true_type{});
            else launch(c0, kp, std::false_type{}, std::true_type{}, std::false_type{});
            return;
          }
        }
        launch(c0, kp, std::false_type{}, std::false_type{}, std::false_type{});
      });
    }
  };
  if (rounded) go(std::true_type{}, std::false_type{});
  else with_flag(relu_bf16, [&](auto kr) { go(std::false_type{}, kr); });
}

// Segment length of the LDS backward: 8 rows when the map's items fit one
// 256-thread block, else 4 while they fit max_items threads; 0 = too many.
// The 4-row walk fits 128 VGPRs, so its blocks may take up to 1024 threads
// (maps up to 128x96 or 256x48): one block per CU, 16 waves.
int box_bwd_lds_seg(int H, int W, int max_items) {
  if (n_chunks(W) * n_segs(H, 8) <= 256) return 8;
  if (n_chunks(W) * n_segs(H, 4) <= max_items) return 4;
  return 0;
}

int box_bwd_lds_waves(int H, int W, int max_items) {
  const int seg = box_bwd_lds_seg(H, W, max_items);
  return seg == 0 ? 0 : (n_chunks(W) * n_segs(H, seg) + 63) / 64;
}

// A call whose maps give fewer than kBwdFillWaves waves with 8-row items
// takes 4-row items instead (twice the waves, each with fewer registers):
// 8 x 64 maps of 64x48 with 8 boxes, 51.5 -> 46.4 us; with 32 x 256 maps the
// 8-row items stay faster (163 against 209 us).
constexpr long kBwdFillWaves = 2048;  // 8 waves on each of 256 CUs
int box_bwd_lds_seg_maps(int H, int W, long maps) {
  const int seg = box_bwd_lds_seg(H, W, kBwdLdsItems);
  if (seg == 8 && maps * ((n_chunks(W) * n_segs(H, 8) + 63) / 64) < kBwdFillWaves &&
      n_chunks(W) * n_segs(H, 4) <= 256)
    return 4;
  return seg;
}

int box_bwd_lds_waves_maps(int H, int W, long maps) {
  const int seg = box_bwd_lds_seg_maps(H, W, maps);
  return seg == 0 ? 0 : (n_chunks(W) * n_segs(H, seg) + 63) / 64;
}

bool box_bwd_lds_computes_taps(int N, int C, int H, int W, int B, int stride) {
  return stride == 1 && W >= kQ && H >= 4 && lds_pitch_class(H, W) > 0 && (long)N * C * B <= kTapsHereBoxes &&
         box_bwd_lds_seg_maps(H, W, (long)N * C) == 4 && H <= box_bwd_lds_waves_maps(H, W, (long)N * C) * 16;
}

hipError_t launch_box_bwd_lds(const float* x, const int* taps, const float* boxes, const float* gy, void* gx, float* partials, int N,
                              int C, int H, int W, int B, bool rounded, bool relu_bf16, int stride, hipStream_t s) {
  if (rounded && relu_bf16) return hipErrorInvalidValue;
  const int seg = box_bwd_lds_seg_maps(H, W, (long)N * C);
  if (seg == 8) bwd_lds_t<8, 256>(x, taps, boxes, gy, gx, partials, N, C, H, W, B, rounded, relu_bf16, stride, s);
  else if (seg == 4 && n_chunks(W) * n_segs(H, 4) <= 256)
    bwd_lds_t<4, 256>(x, taps, boxes, gy, gx, partials, N, C, H, W, B, rounded, relu_bf16, stride, s);
  else if (seg == 4)
    bwd_lds_t<4, kBwdLdsItems>(x, taps, boxes, gy, gx, partials, N, C, H, W, B, rounded, relu_bf16, stride, s);
  else return hipErrorInvalidValue;
  return last_error();
}

}  // namespace bc
