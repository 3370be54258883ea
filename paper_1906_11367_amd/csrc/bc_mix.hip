// 1x1 mix over the C*B filtered maps (Section 1 and 3.2 of the paper: the
// depthwise box filters are followed by a 1x1 convolution), as MFMA GEMMs on
// gfx950.  Per image n with P = H*W pixels:
//   FWD        out[n] (M x P) = w (M x K)   * in[n] (K x P)
//   BWD_DATA   out[n] (K x P) = w^T (K x M) * grad[n] (M x P)
//   BWD_WEIGHT out   (M x K) = sum_n grad[n] (M x P) * in[n]^T (P x K)
// One kernel template covers the three: C(i, j) = sum_l A(i, l) * B(l, j)
// with A and B either contiguous along the reduction index l ("KC") or along
// their row/column index.  Tiles are staged through LDS in l-contiguous
// layout (transposed on the way in where needed) and fed to
// v_mfma_f32_32x32x16_bf16 (bf16 operands) or v_mfma_f32_32x32x2_f32.
#include "bc_common.hpp"
#include "bc_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace bc {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

// Block tiles are kTile x kTile, kTile = 128 or 64: 4 waves in a 2 x 2
// arrangement of sub-tiles of half the side (mix_tile chooses).
constexpr int kMixThreads = 256;

// Storage dtype codes follow bc_dtype: 0 = int32, 1 = fp32, 2 = bf16.
template <int DT> struct StoreBytes { static constexpr int v = DT == 2 ? 2 : 4; };

// Raw storage bits of one element.
template <int DT>
__device__ __forceinline__ uint32_t ld_bits(const char* base, size_t idx) {
  if constexpr (DT == 2) return reinterpret_cast<const uint16_t*>(base)[idx];
  else return reinterpret_cast<const uint32_t*>(base)[idx];
}

// Loaded data is kept in registers as loaded, in vectors of the load's width:
// the values of a load in flight then stay one register tuple, where words
// taken apart are copied out of it, which waits for the load.
template <int N> using Words = uint32_t __attribute__((ext_vector_type(N)));

// N words from memory of the element type's own alignment (2 or 4 bytes): one
// wide load, which global memory accesses may be at any alignment here, so
// that rows of an odd length cost no more instructions than aligned ones.
template <int N, int kAlign> struct __attribute__((packed, aligned(kAlign))) Bytes { uint32_t w[N]; };

template <int DT, int N>
__device__ __forceinline__ Words<N> ld_wide(const char* base, size_t idx) {
  return __builtin_bit_cast(Words<N>, *reinterpret_cast<const Bytes<N, StoreBytes<DT>::v>*>(base + idx * StoreBytes<DT>::v));
}

// The same N words element by element, elements from `avail` on 0: for the
// last elements of an operand, which a wide load would run past.
template <int DT, int N>
__device__ __forceinline__ Words<N> ld_few(const char* base, size_t idx, int avail) {
  Words<N> w;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    if constexpr (DT == 2) {
      const uint32_t lo = 2 * k < avail ? ld_bits<DT>(base, idx + 2 * k) : 0u;
      const uint32_t hi = 2 * k + 1 < avail ? ld_bits<DT>(base, idx + 2 * k + 1) : 0u;
      w[k] = lo | (hi << 16);
    } else {
      w[k] = k < avail ? ld_bits<DT>(base, idx + k) : 0u;
    }
  }
  return w;
}

// N words at element idx, of which `avail` elements lie in the operand;
// `wide`: all of them lie in its memory (whatever row they belong to).
template <int DT, int N>
__device__ __forceinline__ Words<N> ld_run(const char* base, size_t idx, bool wide, int avail) {
  Words<N> w;
  if (wide) w = ld_wide<DT, N>(base, idx);
  else w = ld_few<DT, N>(base, idx, avail);
  return w;
}

// Element k of stored words, as raw bits (bf16 in the low half).
template <int DT, int N>
__device__ __forceinline__ uint32_t word_bits(const Words<N>& w, int k) {
  if constexpr (DT == 2) return (k & 1) ? w[k / 2] >> 16 : w[k / 2] & 0xffffu;
  else return w[k];
}

// Buffer-resource loads: a wave-uniform descriptor of one operand (base and
// byte size, so that the hardware returns zeros past its end), a per-thread
// byte offset and a wave-uniform byte offset.
constexpr int kBufWord3 = 0x00020000;  // raw 32-bit data, no format conversion

template <int N>
__device__ __forceinline__ Words<N> buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  static_assert(N == 2 || N == 4, "8 or 16 bytes");
  if constexpr (N == 4) return __builtin_bit_cast(Words<N>, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
  else return __builtin_bit_cast(Words<N>, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
}

// Storage bits -> fp32 value.
template <int DT>
__device__ __forceinline__ float bits_to_f32(uint32_t b) {
  if constexpr (DT == 0) return (float)(int)b;
  else if constexpr (DT == 1) return __uint_as_float(b);
  else return __uint_as_float(b << 16);
}

// Two fp32 values -> packed bf16 pair (lo in bits 0..15), round to nearest
// even; lowers to one v_cvt_pk_bf16_f32.
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  const __bf16 a = (__bf16)lo, b = (__bf16)hi;
  return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

template <int DT, bool MASK>
__device__ __forceinline__ float operand_f32(uint32_t b, uint32_t m) {
  float f = bits_to_f32<DT>(b);
  if constexpr (MASK) f = (__uint_as_float(m) > 0.f) ? f : 0.f;
  return f;
}

// Element offset of (row r, reduction index l) in a bf16 LDS tile.  The
// 16-byte chunks of a row are XOR-swizzled by (r / 16) % 4: the transposed
// stores (lanes 4 rows apart) and the MFMA operand reads (32 consecutive rows)
// then both hit distinct banks.
template <int PITCH>
__device__ __forceinline__ int bf16_tile_off(int r, int l) {
  constexpr int kChunks = (PITCH - 8) / 8;  // 16-byte chunks per row: 8 (64 deep) or 16 (128 deep)
  static_assert((kChunks & (kChunks - 1)) == 0, "a power of two");
  return r * PITCH + ((((l >> 3) ^ (r >> 4)) & (kChunks - 1)) << 3) + (l & 7);
}

// One GEMM operand X(r, l): rows r in [0, rows), reduction index l in
// [0, depth).  KC: element (r, l) at p[r * ld + l] (l contiguous); otherwise
// at p[l * ld + r] (r contiguous).  Optional fp32 mask with the same indexing:
// elements whose mask is not > 0 read as zero (ReLU derivative).
//
// A block stages rows [r0, r0 + ROWS) x l in [l0, l0 + BK) into an LDS tile
// T[ROWS][PITCH] in the compute type with l contiguous (what the MFMA operand
// registers hold).  Loading (global -> registers, issued a whole K-step ahead)
// is split from storing (registers -> LDS), so the loads of the next tile are
// in flight while the current one feeds the MFMAs.
//   KC:     a unit is UL consecutive l of one row
//   not KC: a unit is UL consecutive l x 4 consecutive r; the 4 x UL block is
//           transposed in registers so every LDS write is 16 contiguous bytes
//           of one row.
// NU units per thread.  bf16 storage without a mask is kept packed and never
// converted.
// kVec: the operand's rows are aligned for wide loads (vec_operand), which
// then serve every tile, those at the operand's edges too.  A kernel takes one
// kind of load or the other: where both write the registers of a tile in
// flight, the compiler joins them by copies that wait for the loads as soon as
// they are issued (fp32, 4 x 128 x 1024 x 65536 in N, M, K, P, both kinds in
// one kernel: FWD 622 us, BWD_DATA 629; one kind each: 546 and 590).
template <bool BF16, int DT, bool KC, bool MASK, int ROWS, int kBK, bool kVec>
struct Stager {
  static constexpr int BK = kBK;
  static constexpr int PITCH = BF16 ? BK + 8 : BK + 1;  // elements; bf16 rows are 16-byte aligned
  static constexpr int UL = BF16 ? 8 : 4;               // l per unit
  static constexpr int NU = KC ? (ROWS * BK / UL) / kMixThreads : (ROWS / 4) * (BK / UL) / kMixThreads;
  static_assert(NU >= 1, "every thread has a unit");
  static constexpr bool kRaw = BF16 && DT == 2 && !MASK;
  static constexpr int SB = StoreBytes<DT>::v;
  // a load: kLW words of kLE elements; kLoads of them per unit (of the mask:
  // always 4 words, kMaskLoads per unit)
  static constexpr int kLW = KC ? 4 : SB;
  static constexpr int kLE = kLW * 4 / SB;
  static constexpr int kLoads = KC ? UL / kLE : UL;
  static constexpr int kMaskLoads = KC ? UL / 4 : UL;
  using E = typename std::conditional<BF16, uint16_t, float>::type;

  // Byte offset of this thread's first load inside a tile (the same for every
  // K-step); its other loads sit a wave-uniform step further each: KC units
  // are kMixThreads / (BK / UL) rows apart, non-KC rows one l apart (and
  // units kUnitL l apart).
  static constexpr int kUnitL = KC ? 0 : kMixThreads / (ROWS / 4) * UL;

  const char* p;
  const float* mask;
  long ld;
  int rows, depth;
  long extent;  // elements of this image's operand
  int lrem;     // reduction indices left from the loaded tile's first
  uint32_t off0, end, mend;
  __amdgpu_buffer_rsrc_t rs, mrs;
  Words<kLW> v[NU * kLoads];
  Words<4> m[MASK ? NU * kMaskLoads : 1];

  // Offsets, and buffer descriptors covering this image's operand (and mask).
  __device__ __forceinline__ void init_offsets() {
    const int tid = threadIdx.x;
    if constexpr (KC) off0 = (uint32_t)(((long)(tid / (BK / UL)) * ld + (tid % (BK / UL)) * UL) * SB);
    else off0 = (uint32_t)(((long)((tid / (ROWS / 4)) * UL) * ld + (tid % (ROWS / 4)) * 4) * SB);
    extent = KC ? (long)(rows - 1) * ld + depth : (long)(depth - 1) * ld + rows;  // elements
    end = (uint32_t)(extent * SB);
    mend = (uint32_t)(extent * 4);
    rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), (short)0, (int)end, kBufWord3);
    if constexpr (MASK) mrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(mask), (short)0, (int)mend, kBufWord3);
  }

  __device__ __forceinline__ void load(int r0, int l0) {
    lrem = depth - l0;
    if constexpr (kVec) load_vec(r0, l0);
    else load_any(r0, l0);
  }

  // Through the buffer descriptor: the thread's one offset plus a wave-uniform
  // offset per K-step and unit, so no address is computed in the loop, and no
  // branch surrounds a load.  At the operand's edges, what lies past its end
  // reads as 0 (the wave-uniform offset is held to its size, from which the
  // range check subtracts it); rows past the last read the next l's values
  // (row-contiguous) and are not stored; l past the range is zeroed when the
  // tile is stored to LDS.  No load straddles the operand's end: its rows are
  // whole units.
  __device__ __forceinline__ void load_vec(int r0, int l0) {
    const uint32_t origin = (uint32_t)(KC ? (long)r0 * ld + l0 : (long)l0 * ld + r0);
    const uint32_t step = (uint32_t)(KC ? (long)(kMixThreads / (BK / UL)) * ld : ld);  // elements
    const uint32_t moff = off0 / SB * 4;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
#pragma unroll
      for (int e = 0; e < kLoads; ++e) {
        const uint32_t at = KC ? origin + u * step + e * kLE : origin + (u * kUnitL + e) * step;
        v[u * kLoads + e] = buf_ld<kLW>(rs, off0, min(at * SB, end));
      }
      if constexpr (MASK) {
#pragma unroll
        for (int e = 0; e < kMaskLoads; ++e) {
          const uint32_t at = KC ? origin + u * step + e * 4 : origin + (u * kUnitL + e) * step;
          m[u * kMaskLoads + e] = buf_ld<4>(mrs, moff, min(at * 4, mend));
        }
      }
    }
  }

  // Operands of any alignment: the same wide loads from clamped addresses.
  // What lies outside needs no guard where it only reaches outputs that are
  // not stored (rows past the last: the last row again, or, row-contiguous,
  // the next l's values); l past the range is zeroed when the tile is stored
  // to LDS.  Only the operand's last few elements, which a wide load would run
  // past, are read one by one.
  __device__ __forceinline__ void load_any(int r0, int l0) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int unit = tid + u * kMixThreads;
      if constexpr (KC) {
        const int r = min(r0 + unit / (BK / UL), rows - 1), l = l0 + (unit % (BK / UL)) * UL;
        const long row = (long)r * ld;
#pragma unroll
        for (int e = 0; e < kLoads; ++e) {
          const long idx = row + min(l + e * kLE, depth - 1);
          v[u * kLoads + e] = ld_run<DT, kLW>(p, idx, idx + kLE <= extent, depth - l - e * kLE);
        }
        if constexpr (MASK) {
#pragma unroll
          for (int e = 0; e < kMaskLoads; ++e) {
            const long idx = row + min(l + e * 4, depth - 1);
            m[u * kMaskLoads + e] = ld_run<1, 4>(reinterpret_cast<const char*>(mask), idx, idx + 4 <= extent, depth - l - e * 4);
          }
        }
      } else {
        const int r = r0 + (unit % (ROWS / 4)) * 4, lb = l0 + (unit / (ROWS / 4)) * UL;
#pragma unroll
        for (int e = 0; e < UL; ++e) {
          const long idx = (long)min(lb + e, depth - 1) * ld + min(r, rows - 1);
          v[u * UL + e] = ld_run<DT, kLW>(p, idx, idx + 4 <= extent, rows - r);
          if constexpr (MASK) m[u * UL + e] = ld_run<1, 4>(reinterpret_cast<const char*>(mask), idx, idx + 4 <= extent, rows - r);
        }
      }
    }
  }

  // Element k of unit u (KC: l of the unit; else element i of its l = e).
  __device__ __forceinline__ float f_kc(int u, int k) const {
    return operand_f32<DT, MASK>(word_bits<DT, kLW>(v[u * kLoads + k / kLE], k % kLE), MASK ? m[u * kMaskLoads + k / 4][k % 4] : 0u);
  }
  __device__ __forceinline__ float f_rc(int u, int e, int i) const {
    return operand_f32<DT, MASK>(word_bits<DT, kLW>(v[u * kLoads + e], i), MASK ? m[u * kMaskLoads + e][i] : 0u);
  }

  // kTail: the tile reaches past the reduction's end; what lies there is
  // stored as 0.
  template <bool kTail>
  __device__ __forceinline__ void store(E* T) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int unit = tid + u * kMixThreads;
      if constexpr (KC) {
        const int r = unit / (BK / UL), l = (unit % (BK / UL)) * UL, left = lrem - l;
        auto at = [&](int k) { return !kTail || left > k ? f_kc(u, k) : 0.f; };
        if constexpr (BF16) {
          Words<4> q;
          if constexpr (kRaw) {
            q = v[u];
            if constexpr (kTail) {
#pragma unroll
              for (int k = 0; k < 4; ++k) q[k] &= left >= 2 * k + 2 ? 0xffffffffu : left == 2 * k + 1 ? 0xffffu : 0u;
            }
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) q[k] = pack2_bf16(at(2 * k), at(2 * k + 1));
          }
          *reinterpret_cast<Words<4>*>(T + bf16_tile_off<PITCH>(r, l)) = q;
        } else {
          E* dst = T + r * PITCH + l;
#pragma unroll
          for (int k = 0; k < UL; ++k) dst[k] = at(k);
        }
      } else {
        const int r = (unit % (ROWS / 4)) * 4, lb = (unit / (ROWS / 4)) * UL, left = lrem - lb;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          auto at = [&](int e) { return !kTail || left > e ? f_rc(u, e, i) : 0.f; };
          if constexpr (BF16) {
            Words<4> q;
            if constexpr (kRaw) {
              // element i of rows (l, l+1) -> one packed word: bytes of the
              // low (i even) or high (i odd) halves of the two source words
              const uint32_t sel = (i & 1) ? 0x07060302u : 0x05040100u;
#pragma unroll
              for (int k = 0; k < 4; ++k) {
                q[k] = __builtin_amdgcn_perm(v[u * UL + 2 * k + 1][i >> 1], v[u * UL + 2 * k][i >> 1], sel);
                if constexpr (kTail) q[k] &= left >= 2 * k + 2 ? 0xffffffffu : left == 2 * k + 1 ? 0xffffu : 0u;
              }
            } else {
#pragma unroll
              for (int k = 0; k < 4; ++k) q[k] = pack2_bf16(at(2 * k), at(2 * k + 1));
            }
            *reinterpret_cast<Words<4>*>(T + bf16_tile_off<PITCH>(r + i, lb)) = q;
          } else {
            E* dst = T + (r + i) * PITCH + lb;
#pragma unroll
            for (int e = 0; e < UL; ++e) dst[e] = at(e);
          }
        }
      }
    }
  }
};

// Stages the loaded tiles of both operands (the same reduction indices).
template <typename SA, typename SB>
__device__ __forceinline__ void store_tiles(const SA& sa, const SB& sb, typename SA::E* As, typename SB::E* Bs) {
  if (sa.lrem < SA::BK) {
    sa.template store<true>(As);
    sb.template store<true>(Bs);
  } else {
    sa.template store<false>(As);
    sb.template store<false>(Bs);
  }
}

// Stores the TT x TT accumulator tiles of one wave.  OK: 0 = fp32, 1 = int32
// (exact integer values), 3 = fp32 accumulate, 4 = fp32 with ReLU.  `full`
// (block-uniform) skips the bounds checks.  NT: non-temporal stores (0, 1, 4).
template <int OK, bool NT, int TT>
__device__ __forceinline__ void epilogue(const f32x16_t (&acc)[TT][TT], char* cbase, int ib, int jb, int rows,
                                         int cols, long ldc, bool full) {
#pragma unroll
  for (int x = 0; x < TT; ++x)
#pragma unroll
    for (int y = 0; y < TT; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = ib + x * 32 + 8 * (r >> 2) + (r & 3);
        const int j = jb + y * 32;
        if (full || (i < rows && j < cols)) {
          const float v = acc[x][y][r];
          const size_t o = (size_t)i * ldc + j;
          if constexpr (OK == 3) {
            reinterpret_cast<float*>(cbase)[o] += v;
          } else if constexpr (OK == 1) {
            if constexpr (NT) __builtin_nontemporal_store((int)v, reinterpret_cast<int*>(cbase) + o);
            else reinterpret_cast<int*>(cbase)[o] = (int)v;
          } else {
            const float u = OK == 4 ? fmaxf(v, 0.f) : v;
            if constexpr (NT) __builtin_nontemporal_store(u, reinterpret_cast<float*>(cbase) + o);
            else reinterpret_cast<float*>(cbase)[o] = u;
          }
        }
      }
}

// Occupancy target (waves per SIMD) of one GEMM variant.  The kernel is
// bound by global-load latency (one K-step of each operand in flight per
// block), so a third resident block per CU pays whenever the variant still
// fits in 168 registers without spilling -- the accumulators then move from
// AGPRs to VGPRs.  Variants that would spill (l-contiguous masked or fp32
// operands in bf16 compute, the bf16 weight-gradient GEMM) keep two.  Loads from
// clamped addresses (kVec false) take more: where one in flight was spilled, and
// so waited for, 2 x 940 x 763 x 2451 in N, M, K, P, masked, took 145 us instead
// of 56, the weight gradient of 11 x 808 x 8 x 572 18.6 instead of 14.6.
template <bool BF16, int ADT, bool AKC, bool AMASK, int BDT, bool BKC, bool BMASK, int kTile, bool kVec>
constexpr int mix_waves() {
  if (kTile == 64) {
    if (!BF16 || kVec || !(AMASK || BMASK)) return 3;
    return (AKC ? ADT == 1 && BDT == 2 : BDT == 1) ? 3 : 2;
  }
  if (!BF16) return (AKC && AMASK) ? 2 : 3;
  if (AMASK || BMASK) return 2;
  if (AKC && !BKC) return (ADT == 2 && BDT == 2) ? 3 : 2;
  if (!AKC && !BKC) return (ADT == 1 && BDT == 1) || !kVec ? 2 : 3;
  return 2;
}

// out-kind: 0 = store fp32 (relu optional), 1 = store int32 (exact integers),
// 2 = store fp32 partial (BWD_WEIGHT split), 3 = fp32 with accumulate; plus
// kOutNT for non-temporal stores of 0 and 1.
constexpr int kOutNT = 8;

// K-step depth.  bf16 storage on both operands, both contiguous along the
// reduction (BWD_WEIGHT): 128, so that each operand row is read as 256-byte
// runs; 64-wide tiles take twice the depth of 128-wide ones, which keeps a
// unit for every thread and halves the K-steps.
template <bool BF16, int ADT, bool AKC, bool AMASK, int BDT, bool BKC, bool BMASK, int kTile>
constexpr int mix_depth() {
  if (kTile == 64) return BF16 ? 128 : 64;
  if (BF16 && AKC && BKC && !AMASK && !BMASK && ADT == 2 && BDT == 2) return 128;
  return BF16 ? 64 : 32;
}

template <bool BF16, int ADT, bool AKC, bool AMASK, int BDT, bool BKC, bool BMASK, int kTile, bool kVecA, bool kVecB>
__global__ __launch_bounds__(kMixThreads)
__attribute__((amdgpu_waves_per_eu(mix_waves<BF16, ADT, AKC, AMASK, BDT, BKC, BMASK, kTile, kVecA && kVecB>(), 8))) void
k_mix_gemm(
    const void* __restrict__ a, const void* __restrict__ b, const float* __restrict__ aux, void* __restrict__ out,
    int rows, int cols, int depth, long lda, long ldb, long ldc, long a_bs, long b_bs, long c_bs,
    int mt, int nt, int zt, int nsplit_p, int pchunk, int out_kind, int relu) {
  constexpr int kDepth = mix_depth<BF16, ADT, AKC, AMASK, BDT, BKC, BMASK, kTile>();
  using SA = Stager<BF16, ADT, AKC, AMASK, kTile, kDepth, kVecA>;
  using SB = Stager<BF16, BDT, BKC, BMASK, kTile, kDepth, kVecB>;
  constexpr int BK = SA::BK, PITCH = SA::PITCH;
  constexpr int TT = kTile / 64, kSub = kTile / 2;  // 32 x 32 tiles and rows per wave, each way
  using E = typename SA::E;
  __shared__ __align__(16) E As[kTile * PITCH];
  __shared__ __align__(16) E Bs[kTile * PITCH];

  // logical tile id: XCD-contiguous, row tiles fastest (blocks sharing one B
  // tile run together on one XCD)
  const int total = mt * nt * zt;
  const int per = gridDim.x >> 3;
  const int L = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (L >= total) return;
  const int tm = L % mt, tn = (L / mt) % nt, z = L / (mt * nt);

  // batch item and reduction range of this block
  int n = z, l_begin = 0, l_end = depth;
  if (nsplit_p > 0) {  // BWD_WEIGHT: z = n * nsplit_p + sp
    n = z / nsplit_p;
    const int sp = z - n * nsplit_p;
    l_begin = sp * pchunk;
    l_end = min(depth, l_begin + pchunk);
  }
  SA sa;
  sa.p = reinterpret_cast<const char*>(a) + (size_t)n * a_bs * StoreBytes<ADT>::v;
  sa.mask = AMASK ? aux + (size_t)n * a_bs : nullptr;
  sa.ld = lda; sa.rows = rows; sa.depth = depth;
  SB sb;
  sb.p = reinterpret_cast<const char*>(b) + (size_t)n * b_bs * StoreBytes<BDT>::v;
  sb.mask = BMASK ? aux + (size_t)n * b_bs : nullptr;
  sb.ld = ldb; sb.rows = cols; sb.depth = depth;
  sa.init_offsets();
  sb.init_offsets();
  // loads stop at this block's reduction range (a split chunk need not be a
  // whole number of K-steps; the descriptors keep the operand's extent)
  sa.depth = l_end;
  sb.depth = l_end;

  const int i0 = tm * kTile, j0 = tn * kTile;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  f32x16_t acc[TT][TT];
#pragma unroll
  for (int x = 0; x < TT; ++x)
#pragma unroll
    for (int y = 0; y < TT; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  if (l_begin < l_end) {
    sa.load(i0, l_begin);
    sb.load(j0, l_begin);
    store_tiles(sa, sb, As, Bs);
    __syncthreads();
  }
  for (int l0 = l_begin; l0 < l_end; l0 += BK) {
    const bool more = l0 + BK < l_end;
    if (more) {  // next tile's loads in flight during this tile's MFMAs
      sa.load(i0, l0 + BK);
      sb.load(j0, l0 + BK);
    }
    if constexpr (BF16) {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 16) {
        bf16x8_t af[TT], bfr[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          af[t] = *reinterpret_cast<const bf16x8_t*>(As + bf16_tile_off<PITCH>(wm * kSub + t * 32 + (lane & 31), kk + 8 * (lane >> 5)));
          bfr[t] = *reinterpret_cast<const bf16x8_t*>(Bs + bf16_tile_off<PITCH>(wn * kSub + t * 32 + (lane & 31), kk + 8 * (lane >> 5)));
        }
#pragma unroll
        for (int x = 0; x < TT; ++x)
#pragma unroll
          for (int y = 0; y < TT; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[x], bfr[y], acc[x][y], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 2) {
        float af[TT], bfr[TT];
#pragma unroll
        for (int t = 0; t < TT; ++t) {
          af[t] = As[(wm * kSub + t * 32 + (lane & 31)) * PITCH + kk + (lane >> 5)];
          bfr[t] = Bs[(wn * kSub + t * 32 + (lane & 31)) * PITCH + kk + (lane >> 5)];
        }
#pragma unroll
        for (int x = 0; x < TT; ++x)
#pragma unroll
          for (int y = 0; y < TT; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(af[x], bfr[y], acc[x][y], 0, 0, 0);
      }
    }
    __syncthreads();
    if (more) {
      store_tiles(sa, sb, As, Bs);
      __syncthreads();
    }
  }

  // Epilogue.  Accumulator element r of lane t in a 32 x 32 tile is
  // C[8 * (r / 4) + 4 * (t / 32) + r % 4][t % 32].
  char* cbase = reinterpret_cast<char*>(out) + (size_t)z * c_bs * 4;
  const bool full = i0 + kTile <= rows && j0 + kTile <= cols;
  const int ib = i0 + wm * kSub + 4 * (lane >> 5), jb = j0 + wn * kSub + (lane & 31);
  switch (out_kind) {
    case 1: epilogue<1, false>(acc, cbase, ib, jb, rows, cols, ldc, full); break;
    case 1 | kOutNT: epilogue<1, true>(acc, cbase, ib, jb, rows, cols, ldc, full); break;
    case 3: epilogue<3, false>(acc, cbase, ib, jb, rows, cols, ldc, full); break;
    case kOutNT:
      if (relu) epilogue<4, true>(acc, cbase, ib, jb, rows, cols, ldc, full);
      else epilogue<0, true>(acc, cbase, ib, jb, rows, cols, ldc, full);
      break;
    default:
      if (relu) epilogue<4, false>(acc, cbase, ib, jb, rows, cols, ldc, full);
      else epilogue<0, false>(acc, cbase, ib, jb, rows, cols, ldc, full);
  }
}

// ---------------------------------------------------------------------------
// BWD_DATA in bf16, one block per column strip
// ---------------------------------------------------------------------------
// out[n] (K x P) = w^T (K x M) * grad[n] (M x P).  The reduction (the mix's
// M output channels) is short and the output (K rows) is the widest tensor
// of the layer, so the 128 x 128 tiles above spend most of their time on
// exposed load latency: each tile has only M / 64 K-steps.  Here a block
// owns kStripP columns of one image instead: it converts grad[n][:, strip]
// to bf16 once, into LDS in B-operand order (rows p, reduction m contiguous),
// and each wave then produces 64 output rows at a time with no further
// barrier, reading its A operand (w transposed, written in MFMA operand
// order by k_wt_frags) from L2 a group of m-steps ahead, and storing each
// finished 64 x 64 tile while the next one's MFMAs run.  The MFMA sequence
// of every output element is the one k_mix_gemm issues (m ascending in
// steps of 16), so both kernels give the same bits.
constexpr int kStripP = 64;     // output columns per block
constexpr int kWtGroup = 4;     // m-steps of 16 loaded together (one group ahead)

// Fragment count of w^T: K rounded up to 64 rows (two 32-row A fragments per
// wave tile), M to kWtGroup m-steps of 16.
__host__ __device__ __forceinline__ int wt_ksteps(int K) { return ((K + 63) / 64) * 2; }
__host__ __device__ __forceinline__ int wt_msteps(int M) { return ((M + 16 * kWtGroup - 1) / (16 * kWtGroup)) * kWtGroup; }

// w [M][K] -> A fragments of w^T: fragment (kb, ms) is 64 lanes x 8 bf16,
// lane l holding w[16 ms + 8 (l / 32) + e][32 kb + l % 32], e = 0..7 (zero
// outside w), stored at frags[(kb * msteps + ms) * 64 + l].
template <int ADT>
__global__ void k_wt_frags(const void* __restrict__ w, int M, int K, int msteps, size_t total,
                           uint4* __restrict__ frags) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  const int lane = (int)(i & 63);
  const size_t f = i >> 6;
  const int ms = (int)(f % msteps), kb = (int)(f / msteps);
  const int k = kb * 32 + (lane & 31), m0 = ms * 16 + 8 * (lane >> 5);
  uint32_t h[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int m = m0 + e;
    const bool in = m < M && k < K;
    const size_t idx = in ? (size_t)m * K + k : 0;
    if constexpr (ADT == 2) h[e] = in ? (uint32_t)reinterpret_cast<const uint16_t*>(w)[idx] : 0u;
    else h[e] = in ? (pack2_bf16(reinterpret_cast<const float*>(w)[idx], 0.f) & 0xffffu) : 0u;
  }
  frags[i] = make_uint4(h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16));
}

// Elements `by` (0 .. 3) and after of a run moved to its front, zeros after them.
__device__ __forceinline__ void shift_run(uint32_t (&w)[4], int by) {
  const bool one = by & 1, two = by & 2;
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = one ? (i < 3 ? w[i + 1] : 0u) : w[i];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = two ? (i < 2 ? w[i + 2] : 0u) : w[i];
}

// The gradient is staged by loads that no branch surrounds, all 8 of a unit in
// flight: a branch for the operand's end makes the compiler wait for each load
// before the next (12 x 136 x 8 x 65536 in N, M, K, P, fp32 gradient: 197 us,
// 117 without).  kVec (rows of whole runs of 4): through a descriptor, whose
// range check gives zeros past the operand's end.  Else from addresses held
// back to the last whole run, whose elements are moved to their places.
template <int BDT, bool BMASK, bool kVec>
__global__ __launch_bounds__(kMixThreads) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_mix_bwd_data_strip(const uint4* __restrict__ frags,
                                                                    const void* __restrict__ g,
                                                                    const float* __restrict__ aux,
                                                                    float* __restrict__ out, int M, int K, int P,
                                                                    int msteps, int nstrips) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  uint16_t* Bs = reinterpret_cast<uint16_t*>(smem_raw);
  const int pitch = msteps * 16 + 8;   // bf16 elements; rows 16-byte aligned, 4 banks apart
  const int strip = blockIdx.x % nstrips, n = blockIdx.x / nstrips;
  const int p0 = strip * kStripP;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t plane = (size_t)M * P;

  // grad[n][m][p0 + j] -> Bs[j * pitch + m]: units of 8 m x 4 p, transposed
  // in registers so each LDS write is 16 contiguous bytes of one row.  Columns
  // past P hold any values and are not stored; m past M are zeros.
  {
    constexpr int SB = StoreBytes<BDT>::v;  // and the words of a run of 4
    const char* gb = reinterpret_cast<const char*>(g) + (size_t)n * plane * SB;
    const char* mb = BMASK ? reinterpret_cast<const char*>(aux + (size_t)n * plane) : nullptr;
    const uint32_t end = (uint32_t)(plane * SB), mend = (uint32_t)(plane * 4);
    __amdgpu_buffer_rsrc_t gr, mr;
    if constexpr (kVec) gr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(gb), (short)0, (int)end, kBufWord3);
    if constexpr (kVec && BMASK) mr = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(mb), (short)0, (int)mend, kBufWord3);
    const int units = (msteps * 16 / 8) * (kStripP / 4);
    for (int u = tid; u < units; u += kMixThreads) {
      const int pg = u % (kStripP / 4), mg = u / (kStripP / 4);
      const int pp = p0 + pg * 4, m0 = mg * 8;
      Words<SB> raw[8];
      Words<4> mk[BMASK ? 8 : 1];
      int back[8];  // elements the run was held back by
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (kVec) {
          const uint32_t at = (uint32_t)m0 * (uint32_t)P + (uint32_t)pp;
          raw[e] = buf_ld<SB>(gr, at * SB, min((uint32_t)(e * P) * SB, end));
          if constexpr (BMASK) mk[e] = buf_ld<4>(mr, at * 4, min((uint32_t)(e * P) * 4, mend));
        } else {
          const size_t idx = (size_t)min(m0 + e, M - 1) * P + min(pp, P - 1), held = min(idx, plane - 4);
          back[e] = (int)(idx - held);
          raw[e] = ld_wide<BDT, SB>(gb, held);
          if constexpr (BMASK) mk[e] = ld_wide<1, 4>(mb, held);
        }
      }
      uint32_t v[8][4], a[8][4];
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          v[e][i] = word_bits<BDT, SB>(raw[e], i);
          a[e][i] = BMASK ? mk[BMASK ? e : 0][i] : 0u;
        }
      if constexpr (!kVec) {
        int any = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) any |= back[e];
        if (__builtin_amdgcn_ballot_w64(any != 0) != 0) {  // the wave holding the image's last elements
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            shift_run(v[e], back[e]);
            if constexpr (BMASK) shift_run(a[e], back[e]);
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool in = kVec || m0 + e < M;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (BDT != 2 || BMASK) v[e][i] = pack2_bf16(operand_f32<BDT, BMASK>(v[e][i], a[e][i]), 0.f) & 0xffffu;
          if (!in) v[e][i] = 0u;
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint4 q = make_uint4(v[0][i] | (v[1][i] << 16), v[2][i] | (v[3][i] << 16), v[4][i] | (v[5][i] << 16),
                                   v[6][i] | (v[7][i] << 16));
        *reinterpret_cast<uint4*>(Bs + (pg * 4 + i) * pitch + m0) = q;
      }
    }
  }
  __syncthreads();

  // wave tiles: rows [64 (wave + 4 t), + 64) for t = 0, 1, ...; all 64 columns
  const int ntile = (K + 63) / 64;
  const int mytiles = ntile > wave ? (ntile - wave + 3) / 4 : 0;
  const int ngroups = msteps / kWtGroup;
  const int total = mytiles * ngroups;
  // Fragment loads and output stores go through buffer descriptors: one
  // per-lane offset plus a wave-uniform offset each, so the 8 loads of a
  // group and the 64 stores of a tile keep no per-element addresses in
  // registers.
  const __amdgpu_buffer_rsrc_t fr = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint4*>(frags), (short)0,
                                                                      (int)((size_t)wt_ksteps(K) * msteps * 1024), kBufWord3);
  const __amdgpu_buffer_rsrc_t orr = __builtin_amdgcn_make_buffer_rsrc(out + (size_t)n * K * P, (short)0,
                                                                       (int)((size_t)K * P * 4), kBufWord3);
  auto load_group = [&](int t, Words<4> (&a)[kWtGroup][2]) {
    const int kb = 2 * (wave + 4 * (t / ngroups));
    const int ms0 = (t % ngroups) * kWtGroup;
#pragma unroll
    for (int s = 0; s < kWtGroup; ++s)
#pragma unroll
      for (int x = 0; x < 2; ++x) a[s][x] = buf_ld<4>(fr, (uint32_t)lane * 16, (uint32_t)(((kb + x) * msteps + ms0 + s) * 1024));
  };
  f32x16_t acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  const uint16_t* brow = Bs + (lane & 31) * pitch + 8 * (lane >> 5);
  float* obase = out + (size_t)n * K * P;
  // the MFMAs of group t (m-steps of one tile), then the tile's store when
  // it is the tile's last group
  auto step = [&](int t, const Words<4> (&a)[kWtGroup][2]) {
    const int ms0 = (t % ngroups) * kWtGroup;
#pragma unroll
    for (int s = 0; s < kWtGroup; ++s) {
      bf16x8_t bf[2];
#pragma unroll
      for (int y = 0; y < 2; ++y)
        bf[y] = *reinterpret_cast<const bf16x8_t*>(brow + y * 32 * pitch + (ms0 + s) * 16);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const bf16x8_t af = __builtin_bit_cast(bf16x8_t, a[s][x]);
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bf[y], acc[x][y], 0, 0, 0);
      }
    }
    if (t % ngroups != ngroups - 1) return;
    const int i0 = 64 * (wave + 4 * (t / ngroups));
    const int ib = i0 + 4 * (lane >> 5), jb = p0 + (lane & 31);
    if (i0 + 64 <= K && p0 + kStripP <= P) {
      const uint32_t vo = (uint32_t)(ib * P + jb) * 4;
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[x][y][r]), orr, (int)vo,
                                                  ((x * 32 + 8 * (r >> 2) + (r & 3)) * P + y * 32) * 4, 2);
    } else {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int i = ib + x * 32 + 8 * (r >> 2) + (r & 3), j = jb + y * 32;
            if (i < K && j < P) __builtin_nontemporal_store(acc[x][y][r], obase + (size_t)i * P + j);
          }
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  };
  // groups alternate between two register sets, each loaded one group ahead
  Words<4> a0[kWtGroup][2], a1[kWtGroup][2];
  if (total > 0) load_group(0, a0);
  for (int t = 0; t < total; t += 2) {
    if (t + 1 < total) load_group(t + 1, a1);
    step(t, a0);
    if (t + 1 >= total) break;
    if (t + 2 < total) load_group(t + 2, a0);
    step(t + 1, a1);
  }
}

// LDS bytes of the strip kernel's B operand, or 0 where it does not apply.
static size_t strip_lds_bytes(int M) {
  const size_t b = (size_t)kStripP * (wt_msteps(M) * 16 + 8) * 2;
  return b <= (64u << 10) ? b : 0;
}

static size_t wt_frag_bytes(int M, int K) { return (size_t)wt_ksteps(K) * wt_msteps(M) * 64 * 16; }

// dst[i] = bf16(src[i]), round to nearest even, 8 elements per thread.
__global__ void k_cast_bf16(const float* __restrict__ src, uint16_t* __restrict__ dst, size_t n) {
  const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (i + 8 <= n) {
    const float4 a = *reinterpret_cast<const float4*>(src + i);
    const float4 b = *reinterpret_cast<const float4*>(src + i + 4);
    uint4 q;
    q.x = pack2_bf16(a.x, a.y); q.y = pack2_bf16(a.z, a.w);
    q.z = pack2_bf16(b.x, b.y); q.w = pack2_bf16(b.z, b.w);
    *reinterpret_cast<uint4*>(dst + i) = q;
  } else {
    for (size_t k = i; k < n; ++k) dst[k] = (uint16_t)(pack2_bf16(src[k], 0.f) & 0xffffu);
  }
}

hipError_t launch_cast_bf16(const float* src, void* dst, size_t n, hipStream_t s) {
  const size_t threads = (n + 7) / 8;
  hipLaunchKernelGGL(k_cast_bf16, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, src, (uint16_t*)dst, n);
  return hipGetLastError();
}

// ReLU backward of the mix in its compute type: dst[i] = bf16(aux[i] > 0 ?
// g[i] : 0), round to nearest even, 8 elements per thread.  These are the
// operand bits a masked bf16 GEMM (MASK) forms from g and aux on load, so
// the unmasked GEMMs on dst compute exactly the same sums.
__global__ void k_relu_cast_bf16(const float* __restrict__ g, const float* __restrict__ aux,
                                 uint16_t* __restrict__ dst, size_t n) {
  const size_t i = ((size_t)blockIdx.x * blockDim.x + threadIdx.x) * 8;
  if (i >= n) return;
  if (i + 8 <= n) {
    const float4 a0 = *reinterpret_cast<const float4*>(g + i);
    const float4 a1 = *reinterpret_cast<const float4*>(g + i + 4);
    const float4 m0 = *reinterpret_cast<const float4*>(aux + i);
    const float4 m1 = *reinterpret_cast<const float4*>(aux + i + 4);
    uint4 q;
    q.x = pack2_bf16(m0.x > 0.f ? a0.x : 0.f, m0.y > 0.f ? a0.y : 0.f);
    q.y = pack2_bf16(m0.z > 0.f ? a0.z : 0.f, m0.w > 0.f ? a0.w : 0.f);
    q.z = pack2_bf16(m1.x > 0.f ? a1.x : 0.f, m1.y > 0.f ? a1.y : 0.f);
    q.w = pack2_bf16(m1.z > 0.f ? a1.z : 0.f, m1.w > 0.f ? a1.w : 0.f);
    *reinterpret_cast<uint4*>(dst + i) = q;
  } else {
    for (size_t k = i; k < n; ++k) dst[k] = (uint16_t)(pack2_bf16(aux[k] > 0.f ? g[k] : 0.f, 0.f) & 0xffffu);
  }
}

hipError_t launch_relu_cast_bf16(const float* g, const float* aux, void* dst, size_t n, hipStream_t s) {
  const size_t threads = (n + 7) / 8;
  hipLaunchKernelGGL(k_relu_cast_bf16, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, s, g, aux,
                     (uint16_t*)dst, n);
  return hipGetLastError();
}

// Fixed-order sum of split-K partials: out = (accumulate ? out : 0) + sum_s part[s].
__global__ void k_mix_reduce(const float* __restrict__ part, int S, size_t n, float* __restrict__ out, int accumulate) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float s = accumulate ? out[i] : 0.f;
  for (int k = 0; k < S; ++k) s += part[(size_t)k * n + i];
  out[i] = s;
}

// The same sum, four consecutive outputs per thread (n a multiple of 4), the
// partials' loads unrolled so that several are in flight; each output's
// additions keep their order, so the bits are those of k_mix_reduce.
__global__ void k_mix_reduce4(const float4* __restrict__ part, int S, size_t n4, float4* __restrict__ out,
                              int accumulate) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  float4 s = accumulate ? out[i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
  for (int k = 0; k < S; ++k) {
    const float4 p = part[(size_t)k * n4 + i];
    s.x += p.x;
    s.y += p.y;
    s.z += p.z;
    s.w += p.w;
  }
  out[i] = s;
}

// The same for few outputs of many partials, where a thread per output leaves
// the chip idle (48 x 128 outputs of 512 partials: 6 blocks, 27 us): a block
// takes 16 outputs, 16 threads each summing every 16th partial, combined in a
// fixed order.
constexpr size_t kReduceFew = 65536;
__global__ __launch_bounds__(256) void k_mix_reduce_few(const float4* __restrict__ part, int S, size_t n4,
                                                        float4* __restrict__ out, int accumulate) {
  __shared__ float4 red[16][16];
  const int j = threadIdx.x & 15, g = threadIdx.x >> 4;
  const size_t i = (size_t)blockIdx.x * 16 + j;
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (i < n4) {
#pragma unroll 4
    for (int k = g; k < S; k += 16) {
      const float4 p = part[(size_t)k * n4 + i];
      s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
  }
  red[g][j] = s;
  __syncthreads();
  if (g == 0 && i < n4) {
    float4 t = accumulate ? out[i] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const float4 p = red[k][j];
      t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
    }
    out[i] = t;
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Whether a GEMM of rows x cols outputs over zt images is small: 128-wide tiles
// would leave CUs without a block or spend a third of their rows on padding.
constexpr long kMixFillBlocks = 512;  // two on each of 256 CUs
static bool mix_small(int rows, int cols, long zt, long fill = kMixFillBlocks) {
  const long t128 = (long)((rows + 127) / 128) * ((cols + 127) / 128);
  const long t64 = (long)((rows + 63) / 64) * ((cols + 63) / 64);
  return t128 * zt < fill || 3 * t64 <= 8 * t128;
}

// Tile side of such a GEMM: 64 where it is small.  A reduction of one 128-wide
// K-step at most fills half of the twice as deep step of the 64-wide tiles, so
// there one block per CU is enough for the others (int32, 21 x 120 x 8 x 3072 in
// N, M, K, P, 504 128-wide tiles: 13.0 us with those, 17.9 with 64-wide ones; 126
// of them or fewer: 0.7 of the time with 64-wide tiles).  In fp32 two whole
// steps of 32 are as good on the wide tiles (50 x 100 x 64 x 1024, 400 of them:
// 13.7 and 17.2), a second one of 31 is not (30 x 256 x 63 x 1000: 21.3 and 17.7).
static bool mix_shallow_f32(int depth) { return depth <= 32 || depth == 64; }
// Not so for int32, converted on its way (16 x 136 x 64 x 1903: 17.4 and 14.1).
template <bool BF16>
static int mix_tile(int rows, int cols, long zt, int depth, bool i32 = false) {
  const bool shallow = BF16 ? depth <= 64 : i32 ? depth <= 32 : mix_shallow_f32(depth);
  return mix_small(rows, cols, zt, shallow ? kMixFillBlocks / 2 : kMixFillBlocks) ? 64 : 128;
}

struct WeightSplit { int tile, sp, chunk, S; };

static WeightSplit weight_split(int N, int M, int K, int P, bool bf16) {
  const int BK = bf16 ? 64 : 32;
  const int tile = 3L * ((M + 63) / 64) * ((K + 63) / 64) <= 8L * ((M + 127) / 128) * ((K + 127) / 128) ? 64 : 128;
  const long tiles = (long)((M + tile - 1) / tile) * ((K + tile - 1) / tile);
  const int max_sp = (P + BK - 1) / BK;
  int sp = (int)std::min<long>(512, (512 + tiles * N - 1) / (tiles * N));
  if (sp < 1) sp = 1;
  if (sp > max_sp) sp = max_sp;
  int chunk = (P + sp - 1) / sp;
  chunk = ((chunk + BK - 1) / BK) * BK;
  sp = (P + chunk - 1) / chunk;
  return {tile, sp, chunk, N * sp};
}

size_t mix_workspace_bytes(int mode, int N, int M, int K, int P, int compute_dt) {
  if (mode == 1)
    return (compute_dt == 2 && strip_lds_bytes(M) > 0 && (size_t)K * P * 4 < ((size_t)1 << 31)) ? wt_frag_bytes(M, K) : 0;
  if (mode != 2) return 0;
  const WeightSplit ws = weight_split(N, M, K, P, compute_dt == 2);
  return ws.S > 1 ? (size_t)ws.S * M * K * sizeof(float) : 0;
}

// Whether an operand (see Stager) of rows x depth takes the aligned loads: rows
// of whole 16-byte units, and offsets, up to a tile past the end, that fit the
// descriptor's 32 bits.  Images then start aligned too: their stride is whole
// rows.
static bool vec_operand(const void* p, const void* mask, bool kc, long ld, int rows, int depth) {
  if ((ld & 7) || ((uintptr_t)p & 15) || (mask && ((uintptr_t)mask & 15))) return false;
  const long n = kc ? rows : depth;
  return n * ld * 4 < (1L << 31) && (n + 128) * ld * 4 < (1L << 32);
}

template <bool BF16, int ADT, bool AKC, bool AMASK, int BDT, bool BKC, bool BMASK>
static void gemm_launch(int tile, const void* a, const void* b, const float* aux, void* out, int rows, int cols,
                        int depth, long lda, long ldb, long ldc, long a_bs, long b_bs, long c_bs, int zt,
                        int nsplit_p, int pchunk, int out_kind, int relu, hipStream_t s) {
  const int mt = (rows + tile - 1) / tile, nt = (cols + tile - 1) / tile;
  const int total = mt * nt * zt;
  const int grid = (total + 7) & ~7;
  const bool va = vec_operand(a, AMASK ? aux : nullptr, AKC, lda, rows, depth);
  const bool vb = vec_operand(b, BMASK ? aux : nullptr, BKC, ldb, cols, depth);
  auto go = [&](auto kt, auto ka, auto kb) {
    hipLaunchKernelGGL((k_mix_gemm<BF16, ADT, AKC, AMASK, BDT, BKC, BMASK, decltype(kt)::value, decltype(ka)::value,
                                   decltype(kb)::value>),
                       dim3(grid), dim3(kMixThreads), 0, s, a, b, aux, out, rows, cols, depth, lda, ldb, ldc, a_bs, b_bs,
                       c_bs, mt, nt, zt, nsplit_p, pchunk, out_kind, relu);
  };
  auto vec = [&](auto kt) {
    if constexpr (AKC && BKC) {  // both rows have the reduction's length
      if (va && vb) go(kt, std::true_type{}, std::true_type{});
      else go(kt, std::false_type{}, std::false_type{});
    } else {
      if (va && vb) go(kt, std::true_type{}, std::true_type{});
      else if (va) go(kt, std::true_type{}, std::false_type{});
      else if (vb) go(kt, std::false_type{}, std::true_type{});
      else go(kt, std::false_type{}, std::false_type{});
    }
  };
  if (tile == 64) vec(std::integral_constant<int, 64>{});
  else vec(std::integral_constant<int, 128>{});
}

// f(integral_constant dtype) for the stored type of a bf16 operand: fp32 or bf16.
template <typename F>
static void with_dt(int dt, F&& f) {
  if (dt == 2) f(std::integral_constant<int, 2>{});
  else f(std::integral_constant<int, 1>{});
}

// f(a's, b's) for the stored types a GEMM is compiled for: bf16 compute reads
// fp32 or bf16 storage, fp32 compute reads fp32, or (FWD) int32, on both sides.
template <bool BF16, bool kInts, typename F>
static void with_dts(int a_dt, int b_dt, F&& f) {
  if constexpr (BF16) {
    with_dt(a_dt, [&](auto ad) { with_dt(b_dt, [&](auto bd) { f(ad, bd); }); });
  } else {
    if constexpr (kInts) {
      if (a_dt == 0) {
        f(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
        return;
      }
    }
    f(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
  }
}

// Non-temporal stores of the final outputs, per mode: they are read once, by
// a later call, and are larger than the caches; keeping them out leaves the
// caches to the operands the other calls re-read.  Measured on the whole
// layer step (each alone on one GEMM gains less): pose layer 0.657 ->
// 0.638 ms, six stacked layers with ReLU 4.64 -> 4.47 ms.  Run back to back
// with warm caches the GEMMs gain far more (BWD_DATA 171 -> 119 us), and
// after a cache flush they lose (165 -> 186 us): the step is what counts.
constexpr bool kNtFwd = true;
constexpr bool kNtBwdData = true;

template <bool BF16>
static hipError_t launch_mix_t(int mode, const void* a, int a_dt, const void* b, int b_dt, void* out, int out_dt,
                               int N, int M, int K, int P, int relu, const float* aux, int accumulate, void* ws,
                               hipStream_t s) {
  const int out_kind_plain = out_dt == 0 ? 1 : 0;
  const int ok_fwd = out_kind_plain | (kNtFwd ? kOutNT : 0);
  const int ok_bwd_data = out_kind_plain | (kNtBwdData ? kOutNT : 0);
  if (mode == 0) {
    // C = out[n] (M x P): A = w (row-major M x K), B(l=k, j=p) = in[n][k][p]
    if constexpr (BF16) {
      if (a_dt == 2 && b_dt == 2 && out_dt == 1 && mix_fwd_pipe_takes(a, b, N, M, K, P))
        return launch_mix_fwd_pipe(a, b, (float*)out, N, M, K, P, relu, s);
    }
    if constexpr (!BF16) {
      if (a_dt == 1 && b_dt == 1 && out_dt == 1 &&
          mix_small(M, P, N, K == 64 ? kMixFillBlocks / 2 : kMixFillBlocks) &&
          mix_f32_direct_takes(true, N, M, K, P))
        return launch_mix_f32_direct(true, (const float*)a, (const float*)b, nullptr, (float*)out, N, M, K, P, relu, s);
    }
    with_dts<BF16, true>(a_dt, b_dt, [&](auto ad, auto bd) {
      gemm_launch<BF16, decltype(ad)::value, true, false, decltype(bd)::value, false, false>(
          mix_tile<BF16>(M, P, N, K, a_dt == 0), a, b, nullptr, out, M, P, K, K, P, P, 0, (long)K * P, (long)M * P, N, 0, 0, ok_fwd, relu, s);
    });
    return hipGetLastError();
  }
  // (an image of fewer than 4 gradient values holds no whole run: below)
  if (mode == 1 && BF16 && strip_lds_bytes(M) > 0 && out_dt == 1 && (size_t)K * P * 4 < ((size_t)1 << 31) &&
      (size_t)M * P >= 4) {
    // strip kernel: w^T in fragment order in the workspace, then one block
    // per (image, kStripP columns)
    const int ms = wt_msteps(M);
    const size_t nfr = (size_t)wt_ksteps(K) * ms * 64;
    with_dt(a_dt, [&](auto ad) {
      hipLaunchKernelGGL(k_wt_frags<decltype(ad)::value>, dim3((unsigned)((nfr + 255) / 256)), dim3(256), 0, s, a, M,
                         K, ms, nfr, (uint4*)ws);
    });
    const int nstrips = (P + kStripP - 1) / kStripP;
    const size_t shm = strip_lds_bytes(M);
    // rows of whole runs, and byte offsets, up to the last m-step, in 32 bits
    const bool vec = (P & 3) == 0 && (size_t)M * P * 4 < ((size_t)1 << 31) && (size_t)ms * 16 * P * 4 < ((size_t)1 << 32);
    auto go = [&](auto bd, auto masked, auto kv) {
      hipLaunchKernelGGL((k_mix_bwd_data_strip<decltype(bd)::value, decltype(masked)::value, decltype(kv)::value>),
                         dim3(N * nstrips), dim3(kMixThreads), shm, s, (const uint4*)ws, b, aux, (float*)out, M, K, P,
                         ms, nstrips);
    };
    with_dt(b_dt, [&](auto bd) {
      auto with_vec = [&](auto masked) {
        if (vec) go(bd, masked, std::true_type{});
        else go(bd, masked, std::false_type{});
      };
      if (relu) with_vec(std::true_type{});
      else with_vec(std::false_type{});
    });
    return hipGetLastError();
  }
  if constexpr (!BF16) {
    if (mode == 1 && a_dt == 1 && b_dt == 1 && out_dt == 1 && mix_f32_direct_takes(false, N, M, K, P))
      return launch_mix_f32_direct(false, (const float*)a, (const float*)b, aux, (float*)out, N, M, K, P, relu, s);
  }
  if (mode == 1) {
    // C = out[n] (K x P): A(i=k, l=m) = w[m][k] (k contiguous), B(l=m, j=p) = grad[n][m][p]
    with_dts<BF16, false>(a_dt, b_dt, [&](auto ad, auto bd) {
      if (relu)
        gemm_launch<BF16, decltype(ad)::value, false, false, decltype(bd)::value, false, true>(
            mix_tile<BF16>(K, P, N, M), a, b, aux, out, K, P, M, K, P, P, 0, (long)M * P, (long)K * P, N, 0, 0, ok_bwd_data, 0, s);
      else
        gemm_launch<BF16, decltype(ad)::value, false, false, decltype(bd)::value, false, false>(
            mix_tile<BF16>(K, P, N, M), a, b, nullptr, out, K, P, M, K, P, P, 0, (long)M * P, (long)K * P, N, 0, 0, ok_bwd_data, 0, s);
    });
    return hipGetLastError();
  }
  // C = out (M x K): A(i=m, l=p) = grad[n][m][p], B(l=p, j=k) = in[n][k][p]; both p-contiguous.
  // The reduction over (n, p) is split over images and p-chunks into fp32
  // partials, summed in a fixed order by k_mix_reduce.
  const WeightSplit sp = weight_split(N, M, K, P, BF16);
  const bool direct = sp.S == 1;
  void* dst = direct ? out : ws;
  const int ok = direct ? (accumulate ? 3 : 0) : 2;
  bool piped = false;
  if constexpr (BF16) {
    if (a_dt == 2 && b_dt == 2 && !relu && !direct && mix_wgrad_pipe_takes(a, b, N, M, K, P)) {
      const hipError_t e = launch_mix_wgrad_pipe(a, b, (float*)ws, N, M, K, P, sp.sp, sp.chunk, s);
      if (e != hipSuccess) return e;
      piped = true;
    }
  }
  if (!piped) with_dts<BF16, false>(a_dt, b_dt, [&](auto ad, auto bd) {
    if (relu)
      gemm_launch<BF16, decltype(ad)::value, true, true, decltype(bd)::value, true, false>(
          sp.tile, a, b, aux, dst, M, K, P, P, P, K, (long)M * P, (long)K * P, direct ? 0 : (long)M * K, sp.S, sp.sp,
          sp.chunk, ok, 0, s);
    else
      gemm_launch<BF16, decltype(ad)::value, true, false, decltype(bd)::value, true, false>(
          sp.tile, a, b, nullptr, dst, M, K, P, P, P, K, (long)M * P, (long)K * P, direct ? 0 : (long)M * K, sp.S, sp.sp,
          sp.chunk, ok, 0, s);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || direct) return e;
  const size_t n = (size_t)M * K;
  if ((n & 3) == 0 && ((uintptr_t)out & 15) == 0 && n / 4 < kReduceFew && sp.S >= 64) {
    const size_t n4 = n / 4;
    hipLaunchKernelGGL(k_mix_reduce_few, dim3((unsigned)((n4 + 15) / 16)), dim3(256), 0, s, (const float4*)ws, sp.S,
                       n4, (float4*)out, accumulate);
  } else if ((n & 3) == 0 && ((uintptr_t)out & 15) == 0) {
    const size_t n4 = n / 4;
    hipLaunchKernelGGL(k_mix_reduce4, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, s, (const float4*)ws, sp.S,
                       n4, (float4*)out, accumulate);
  } else {
    hipLaunchKernelGGL(k_mix_reduce, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const float*)ws, sp.S, n,
                       (float*)out, accumulate);
  }
  return hipGetLastError();
}

hipError_t launch_mix(int mode, const void* a, int a_dt, const void* b, int b_dt, void* out, int out_dt, int N,
                      int M, int K, int P, int compute_dt, int relu, const float* aux, int accumulate, void* ws,
                      size_t ws_bytes, hipStream_t s) {
  (void)ws_bytes;
  if (compute_dt == 2)
    return launch_mix_t<true>(mode, a, a_dt, b, b_dt, out, out_dt, N, M, K, P, relu, aux, accumulate, ws, s);
  return launch_mix_t<false>(mode, a, a_dt, b, b_dt, out, out_dt, N, M, K, P, relu, aux, accumulate, ws, s);
}

}  // namespace bc
