// The fp32 1x1 mix without LDS (gfx950), for calls of few output tiles:
//   FWD       out[n] (M x P) = w (M x K) * in[n] (K x P)
//   BWD_DATA  out[n] (K x P) = w^T (K x M) * grad[n] (M x P)
// The widest tensor (in, or out) should move at memory rate, but the tiled
// kernel (bc_mix.hip) passes both operands through registers and LDS with one
// K-step in flight and two barriers per step, and such calls have few blocks
// or few steps to hide that behind.  In fp32 the operand of a matrix
// instruction is one word per lane, 32 columns of two reduction indices: the
// K x P operand (and w^T) is read from memory in just that layout, as 128-byte
// runs, so every wave loads its own operands kAhead groups ahead and no wave
// waits for another.  FWD, N x M x K x P: 8 x 64 x 512 x 3072 28 -> 21 us (75
// TFLOP/s of the 154 a large product reaches), 8 x 33 x 500 x 4000 36 -> 21,
// 16 x 96 x 400 x 1024 25 -> 17.
#include "bc_common.hpp"
#include "bc_internal.hpp"

#include <type_traits>

namespace bc {
namespace {

typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kGroup = 8;  // reduction indices per group: lane half h takes 4 h .. 4 h + 3

// One wave computes 32 rows x 32 CT columns.  kMask (BWD_DATA): the gradient
// counts where aux > 0.
template <bool kFwd, bool kMask, int CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 8))) void k_mix_f32_direct(
    const float* __restrict__ w, const float* __restrict__ b, const float* __restrict__ aux, float* __restrict__ out,
    int M, int K, int P, int mt, int nt, int total, int relu) {
  constexpr int kAhead = CT == 2 ? 6 : 8;  // groups in flight
  const int rows = kFwd ? M : K, depth = kFwd ? K : M;
  const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // consecutive waves, and blocks of one XCD, take the row tiles of one column tile
  const int per = gridDim.x >> 3;
  const int id = ((blockIdx.x & 7) * per + (blockIdx.x >> 3)) * 4 + wave;
  if (id >= total) return;
  const int tm = id % mt, rest = id / mt, tn = rest % nt, n = rest / nt;
  const int r0 = tm * 32, p0 = tn * 32 * CT;
  const float* bn = b + (size_t)n * depth * P;
  const float* mn = kMask ? aux + (size_t)n * depth * P : nullptr;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(w), (short)0, M * K * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(bn), (short)0, depth * P * 4, 0x00020000);
  const __amdgpu_buffer_rsrc_t rm =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kMask ? mn : bn), (short)0, depth * P * 4, 0x00020000);
  // rows and columns past the last: the last again (not stored)
  const int row = min(r0 + c, rows - 1);
  const int ao = (kFwd ? row * K + 4 * h : 4 * h * K + row) * 4;
  int bo[CT];
#pragma unroll
  for (int y = 0; y < CT; ++y) bo[y] = (4 * h * P + min(p0 + 32 * y + c, P - 1)) * 4;

  struct Group {
    float a[4], b[CT][4], m[kMask ? CT : 1][4];
  };
  auto ld = [](__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  };
  auto load = [&](Group& f, int g) {
    if constexpr (kFwd) {
      const auto q = __builtin_amdgcn_raw_buffer_load_b128(ra, ao, g * (kGroup * 4), 0);
#pragma unroll
      for (int s = 0; s < 4; ++s) f.a[s] = __uint_as_float(q[s]);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) f.a[s] = ld(ra, ao, (g * kGroup + s) * K * 4);
    }
#pragma unroll
    for (int y = 0; y < CT; ++y)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        f.b[y][s] = ld(rb, bo[y], (g * kGroup + s) * P * 4);
        if constexpr (kMask) f.m[y][s] = ld(rm, bo[y], (g * kGroup + s) * P * 4);
      }
  };
  f32x16_t acc[CT];
#pragma unroll
  for (int y = 0; y < CT; ++y)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[y][r] = 0.f;
  auto multiply = [&](Group& f) {
    if constexpr (kMask) {
#pragma unroll
      for (int y = 0; y < CT; ++y)
#pragma unroll
        for (int s = 0; s < 4; ++s) f.b[y][s] = f.m[y][s] > 0.f ? f.b[y][s] : 0.f;
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int y = 0; y < CT; ++y) acc[y] = __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[s], f.b[y][s], acc[y], 0, 0, 0);
  };

  const int ng = depth / kGroup;
  if (ng > 0) {
    Group f[kAhead];
    // group g is loaded while group g - kAhead + 1 is multiplied; past the last
    // whole group the last is loaded again, so that no load hangs on a branch
#pragma unroll
    for (int d = 0; d + 1 < kAhead; ++d) load(f[d], min(d, ng - 1));
    __builtin_amdgcn_sched_barrier(0);  // the loads stay where they are issued
    int g0 = 0;
    for (; g0 + kAhead <= ng; g0 += kAhead) {
#pragma unroll
      for (int d = 0; d < kAhead; ++d) {
        load(f[(d + kAhead - 1) % kAhead], min(g0 + d + kAhead - 1, ng - 1));
        __builtin_amdgcn_sched_barrier(0);
        multiply(f[d]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d + 1 < kAhead; ++d)
      if (g0 + d < ng) multiply(f[d]);
  }
  if (ng * kGroup < depth) {  // the last few reduction indices, element by element, zeros past them
    Group f;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int l = ng * kGroup + 4 * h + s, lc = min(l, depth - 1) - 4 * h;
      const bool in = l < depth;
      const float a = ld(ra, ao + (kFwd ? lc : lc * K) * 4, 0);
      f.a[s] = in ? a : 0.f;
#pragma unroll
      for (int y = 0; y < CT; ++y) {
        const float v = ld(rb, bo[y] + lc * P * 4, 0);
        f.b[y][s] = in ? v : 0.f;
        if constexpr (kMask) f.m[y][s] = ld(rm, bo[y] + lc * P * 4, 0);
      }
    }
    multiply(f);
  }

  // accumulator element r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
  float* o = out + (size_t)n * rows * P;
  const bool full = r0 + 32 <= rows && p0 + 32 * CT <= P;
#pragma unroll
  for (int y = 0; y < CT; ++y)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = r0 + 4 * h + 8 * (r >> 2) + (r & 3), j = p0 + 32 * y + c;
      const float v = kFwd && relu ? fmaxf(acc[y][r], 0.f) : acc[y][r];
      if (full || (i < rows && j < P)) __builtin_nontemporal_store(v, o + (size_t)i * P + j);
    }
}

template <bool kFwd, bool kMask, int CT>
hipError_t go(const float* w, const float* b, const float* aux, float* out, int N, int M, int K, int P, int relu,
              hipStream_t s) {
  const int rows = kFwd ? M : K;
  const int mt = (rows + 31) / 32, nt = (P + 32 * CT - 1) / (32 * CT), total = mt * nt * N;
  const int blocks = (total + 3) / 4;
  hipLaunchKernelGGL((k_mix_f32_direct<kFwd, kMask, CT>), dim3((blocks + 7) & ~7), dim3(256), 0, s, w, b, aux, out,
                     M, K, P, mt, nt, total, relu);
  return hipGetLastError();
}

long tiles32(int rows, int P, int N, int ct) {
  return (long)((rows + 31) / 32) * ((P + 32 * ct - 1) / (32 * ct)) * N;
}

}  // namespace

// FWD: K a multiple of 4 (16-byte runs of w's rows); the caller asks only where
// the tiled kernel would take 64-wide tiles (elsewhere its 128-wide ones reuse
// more: 4 x 128 x 1024 x 65536 in N, M, K, P 546 us tiled, 697 here), and at two
// whole K-steps of those (K = 64) only where one block per CU would not be full
// either (14 x 256 x 64 x 2048, 448 of them: 14.7 us tiled, 22.8 here; 12 x 256 x
// 32 x 2048 11 and 8.6).
// BWD_DATA: where M and K are short, so that the tiled kernel's padding and its
// one or two K-steps cost most (2 x 48 x 128 x 110592 61 us tiled, 47 here; 4 x
// 17 x 96 x 2451 7.9 and 4.2); with more of either the re-reading of the
// gradient costs more (32 x 64 x 128 x 3072 24 and 30, 8 x 64 x 512 x 3072 25
// and 32).
bool mix_f32_direct_takes(bool fwd, int N, int M, int K, int P) {
  const long top = 1L << 31;
  if ((long)M * K * 4 >= top || (long)(fwd ? K : M) * P * 4 >= top || tiles32(fwd ? M : K, P, N, 1) >= top / 64)
    return false;
  return fwd ? K % 4 == 0 : K <= 128 && M <= 48;
}

hipError_t launch_mix_f32_direct(bool fwd, const float* w, const float* b, const float* aux, float* out, int N, int M,
                                 int K, int P, int relu, hipStream_t s) {
  if (!fwd)
    return relu ? go<false, true, 1>(w, b, aux, out, N, M, K, P, 0, s)
                : go<false, false, 1>(w, b, aux, out, N, M, K, P, 0, s);
  // two column tiles a wave reuse w's operand, one spreads over more SIMDs
  // (1024): two, unless that takes a quarter more rounds of column tiles (us with
  // two and with one: 8 x 64 x 512 x 3072, as many rounds, 21 and 27; 51 x 128 x
  // 896 x 1024, 8 rounds and 7, 114 and 142; 1 x 256 x 1024 x 3072, 2 and 1, 35
  // and 22); any more rounds at reductions of 36 to 128, which have less of w to
  // reuse (10 x 256 x 128 x 2048, 6 rounds and 5, 24.4 and 20.8; 20 x 256 x 56 x
  // 1024, 14.7 and 12.5; at 32 the stores decide: 28 x 208 x 32 x 1024 10.8 and 13)
  const long two = 2 * ((tiles32(M, P, N, 2) + 1023) / 1024), one = (tiles32(M, P, N, 1) + 1023) / 1024;
  return 4 * two <= (K > 32 && K <= 128 ? 4 : 5) * one ? go<true, false, 2>(w, b, nullptr, out, N, M, K, P, relu, s)
                    : go<true, false, 1>(w, b, nullptr, out, N, M, K, P, relu, s);
}

}  // namespace bc
