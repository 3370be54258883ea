// The 1x1 mix forward on bf16 operands as a pipelined GEMM (gfx950):
//   out[n] (M x P) = w (M x K) * in[n] (K x P),  w and in stored as bf16.
// What bounds it: in is the widest tensor read (201 MB at 32 images of 1024 x
// 3072) against 51.5 GFLOP, so it should run at the rate memory delivers in.
// The tiled kernel (bc_mix.hip) keeps one K-step in flight per block and
// passes every operand through registers, where it is transposed for LDS: it
// waits on that latency.  Here both operands go from memory straight into a
// ring of LDS stages (buffer loads with LDS destination), two K-steps ahead,
// one barrier per K-step; the K x P operand stays as it is stored (rows k,
// columns contiguous) and is transposed by the LDS read itself
// (ds_read_b64_tr_b16: the 4 x 16 block a 16-lane group addresses, returned
// column by column), and blocks are persistent, so that the ring keeps filling
// across tiles.
#include "bc_common.hpp"
#include "bc_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace bc {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));
#define BC_LDS __attribute__((address_space(3)))

constexpr int kBK = 64;      // reduction indices per stage
constexpr int kStages = 3;   // ring: one being read, two in flight

// Buffer descriptor: reads past `bytes` return 0.
__device__ __forceinline__ i32x4_t buf_desc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  i32x4_t r;
  r.x = __builtin_amdgcn_readfirstlane((int)a);
  r.y = __builtin_amdgcn_readfirstlane((int)(a >> 32));
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;
  return r;
}

// 16 bytes per lane from (desc, voff + soff) to LDS at lds + 16 * lane.  No
// register is written; the wave waits for it by count (wait_loads).
__device__ __forceinline__ void load_to_lds(const i32x4_t& rs, uint32_t voff, uint32_t soff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 1\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               ::"s"(lds), "v"(voff), "s"(rs), "s"(soff)
               : "memory", "m0");
}

// Waits until at most kLeft of the wave's memory operations are pending, and
// for its LDS reads (whose place the loads after the next barrier may take).
template <int kLeft>
__device__ __forceinline__ void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kLeft) : "memory");
}

// 4 consecutive k of one column per lane, from a row-contiguous LDS tile.
__device__ __forceinline__ s16x4_t read_tr(uint32_t lds) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((BC_LDS s16x4_t*)(uintptr_t)lds);
}

// kWM x kWN waves of 64 x 64 outputs: tiles of 64 kWM rows x 64 kWN columns.
//
// LDS stage, operand A (w): rows m of kBK = 64 values (128 bytes); the 16-byte
// chunk c of row m sits at chunk c ^ ((m >> 1) & 7), so that the 16 lanes
// reading one chunk of 16 rows hit all banks.  Operand B (in): rows k of kBN
// columns; the 64-byte granule g of row k sits at g ^ (k & 3) (g within its
// aligned four), so that the four rows a transposed read takes do.  The loads
// write LDS in lane order, so each lane fetches the chunk that belongs there.
template <int kWM, int kWN, bool kRelu>
__global__ __launch_bounds__(64 * kWM * kWN) void k_mix_fwd_pipe(const uint16_t* __restrict__ w,
                                                               const uint16_t* __restrict__ in,
                                                               float* __restrict__ out, int M, int K, int P, int mt,
                                                               int nt, int tiles) {
  constexpr int kWaves = kWM * kWN, kBM = 64 * kWM, kBN = 64 * kWN;
  constexpr int kABytes = kBM * kBK * 2, kBBytes = kBK * kBN * 2, kStage = kABytes + kBBytes;
  constexpr int kALoads = kABytes / 1024 / kWaves, kBLoads = kBBytes / 1024 / kWaves;  // per wave and stage
  constexpr int kLoads = kALoads + kBLoads;
  constexpr int kRowB = kBN * 2, kRowsPerLoad = 1024 / kRowB;  // bytes of a B row, B rows per load
  static_assert(kABytes % (1024 * kWaves) == 0 && kBBytes % (1024 * kWaves) == 0, "whole loads");
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(BC_LDS unsigned char*)smem_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / kWN, wn = wave % kWN;
  const int nk = K / kBK;
  const i32x4_t ra = buf_desc(w, (uint32_t)((size_t)M * K * 2));

  // this block's tiles: blockIdx.x, + gridDim.x, ...; row tiles fastest
  const int first = blockIdx.x, step = gridDim.x;
  const int mine = first < tiles ? (tiles - first + step - 1) / step : 0;
  const int total = mine * nk;  // stages
  if (total == 0) return;

  const int kr = lane * 16 / kRowB;                     // B row within a load
  auto b_chunk = [&](int k) {                           // source 16-byte chunk of this lane's slot in row k
    const int slot = lane % (kRowB / 16);
    return slot ^ ((k & 3) << 2);
  };

  int load_tile = first, load_k = 0, load_slot = 0;
  i32x4_t rb;
  int lm0 = 0, lp0 = 0;
  auto open_tile = [&](int t) {
    const int tm = t % mt, rest = t / mt, tn = rest % nt, n = rest / nt;
    lm0 = tm * kBM;
    lp0 = tn * kBN;
    rb = buf_desc(in + (size_t)n * K * P, (uint32_t)((size_t)K * P * 2));
  };
  open_tile(load_tile);
  auto issue = [&]() {
    const uint32_t base = lds0 + load_slot * kStage;
#pragma unroll
    for (int i = 0; i < kALoads; ++i) {
      const int ld = wave * kALoads + i, r0 = ld * 8;  // rows r0 .. r0 + 7
      const int row = r0 + (lane >> 3);
      const uint32_t c = (uint32_t)((lane & 7) ^ ((row >> 1) & 7));
      // rows past M: the last row again (their outputs are not stored)
      load_to_lds(ra, (uint32_t)min(lm0 + row, M - 1) * (uint32_t)(K * 2) + c * 16, (uint32_t)(load_k * kBK * 2),
                  base + ld * 1024);
    }
#pragma unroll
    for (int i = 0; i < kBLoads; ++i) {
      const int ld = wave * kBLoads + i, k0 = ld * kRowsPerLoad;
      // columns past P: the last eight again
      const uint32_t vb = (uint32_t)(kr * P + min(lp0 + b_chunk(k0 + kr) * 8, P - 8)) * 2;
      load_to_lds(rb, vb, (uint32_t)((load_k * kBK + k0) * P * 2), base + kABytes + ld * 1024);
    }
    load_slot = load_slot + 1 == kStages ? 0 : load_slot + 1;
    if (++load_k == nk) {
      load_k = 0;
      load_tile += step;
      if (load_tile < tiles) open_tile(load_tile);
    }
  };

  // LDS offsets of the fragments this lane reads, within a stage
  const int arow = wm * 64 + (lane & 31);
  const uint32_t a_off = (uint32_t)(arow * 128);
  const int asw = (arow >> 1) & 7;  // rows 32 apart swizzle alike
  // B: 16-lane group g reads rows 8 (g / 2) + (lane % 16) / 4 (+ 4), columns 16 (g & 1) + 4 (lane % 4)
  const int bk = 8 * (lane >> 5) + ((lane & 15) >> 2);
  const int bp = wn * 64 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
  uint32_t b_off[2];
#pragma unroll
  for (int y = 0; y < 2; ++y) {
    const int p = bp + 32 * y;
    b_off[y] = (uint32_t)(kABytes + bk * kRowB + ((((p >> 3) ^ ((bk & 3) << 2)) << 4) | ((p & 7) << 1)));
  }

  f32x16_t acc[2][2];
  auto clear = [&]() {
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  };
  clear();

  int issued = 0;
  for (; issued < kStages - 1 && issued < total; ++issued) issue();
  int k = 0, t = first, slot = 0;
  int stores = 0;  // K-steps for which stores may still be newer than the awaited loads
  for (int s = 0; s < total; ++s) {
    // this stage's loads are done when at most the next stage's are pending
    // (memory operations of a wave complete in order; after a tile's stores
    // the count that allows for them all exceeds the counter, so its limit)
    if (s + 1 < total) {
      if (stores > 0) wait_loads<63>();
      else wait_loads<kLoads>();
    } else {
      wait_loads<0>();
    }
    if (stores > 0) --stores;
    __builtin_amdgcn_s_barrier();
    if (issued < total) { issue(); ++issued; }
    const uint32_t st = lds0 + slot * kStage;
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 16) {
      bf16x8_t af[2], bf[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint32_t c = (uint32_t)((kk / 8 + (lane >> 5)) ^ asw);
        af[x] = *(BC_LDS bf16x8_t*)(uintptr_t)(st + a_off + x * 32 * 128 + c * 16);
      }
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const s16x4_t lo = read_tr(st + b_off[y] + kk * kRowB), hi = read_tr(st + b_off[y] + (kk + 4) * kRowB);
        bf[y] = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[x], bf[y], acc[x][y], 0, 0, 0);
    }
    slot = slot + 1 == kStages ? 0 : slot + 1;
    if (++k < nk) continue;
    // store the tile: accumulator element r of lane l is row 8 (r / 4) + 4 (l
    // / 32) + r % 4, column l % 32 of its 32 x 32 block
    k = 0;
    const int tm = t % mt, rest = t / mt, tn = rest % nt, n = rest / nt;
    const int ib = tm * kBM + wm * 64 + 4 * (lane >> 5), jb = tn * kBN + wn * 64 + (lane & 31);
    float* o = out + (size_t)n * M * P;
    const bool full = tm * kBM + kBM <= M && tn * kBN + kBN <= P;
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = ib + x * 32 + 8 * (r >> 2) + (r & 3), j = jb + y * 32;
          if (full || (i < M && j < P))
            __builtin_nontemporal_store(kRelu ? fmaxf(acc[x][y][r], 0.f) : acc[x][y][r], o + (size_t)i * P + j);
        }
    clear();
    t += step;
    // a whole tile is 64 stores of every wave; of a ragged one the waves make
    // fewer, so it waits for them here
    if (full) stores = kStages - 1;
    else wait_loads<0>();
  }
}

// The weight gradient on bf16 operands the same way:
//   part[z] (M x K) = sum over a range of pixels of grad[n] (M x P) * in[n]^T
// Both operands are contiguous along the reduction, so both take operand A's
// layout above.  One block per (tile, z), z = n * sp + range.
template <int kWM, int kWN>
__global__ __launch_bounds__(64 * kWM * kWN) void k_mix_wgrad_pipe(const uint16_t* __restrict__ grad,
                                                                 const uint16_t* __restrict__ in,
                                                                 float* __restrict__ part, int M, int K, int P, int mt,
                                                                 int nt, int sp, int chunk, int total) {
  constexpr int kWaves = kWM * kWN, kBM = 64 * kWM, kBN = 64 * kWN;
  constexpr int kABytes = kBM * kBK * 2, kBBytes = kBN * kBK * 2, kStage = kABytes + kBBytes;
  constexpr int kALoads = kABytes / 1024 / kWaves, kBLoads = kBBytes / 1024 / kWaves;
  constexpr int kLoads = kALoads + kBLoads;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(BC_LDS unsigned char*)smem_raw;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / kWN, wn = wave % kWN;
  // consecutive tiles of one z read the same pixels: on one XCD
  const int per = gridDim.x >> 3;
  const int L = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (L >= total) return;
  const int tm = L % mt, tn = (L / mt) % nt, z = L / (mt * nt);
  const int n = z / sp, l0 = (z - n * sp) * chunk, nk = (min(P, l0 + chunk) - l0) / kBK;
  const int m0 = tm * kBM, k0 = tn * kBN;
  const i32x4_t ra = buf_desc(grad + (size_t)n * M * P, (uint32_t)((size_t)M * P * 2));
  const i32x4_t rb = buf_desc(in + (size_t)n * K * P, (uint32_t)((size_t)K * P * 2));
  // source offsets of this lane's loads (rows past the last: the last again)
  uint32_t va[kALoads], vb[kBLoads];
#pragma unroll
  for (int i = 0; i < kALoads; ++i) {
    const int row = (wave * kALoads + i) * 8 + (lane >> 3);
    va[i] = (uint32_t)min(m0 + row, M - 1) * (uint32_t)(P * 2) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
  }
#pragma unroll
  for (int i = 0; i < kBLoads; ++i) {
    const int row = (wave * kBLoads + i) * 8 + (lane >> 3);
    vb[i] = (uint32_t)min(k0 + row, K - 1) * (uint32_t)(P * 2) + (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
  }
  auto issue = [&](int s, int slot) {
    const uint32_t base = lds0 + slot * kStage, so = (uint32_t)((l0 + s * kBK) * 2);
#pragma unroll
    for (int i = 0; i < kALoads; ++i) load_to_lds(ra, va[i], so, base + (wave * kALoads + i) * 1024);
#pragma unroll
    for (int i = 0; i < kBLoads; ++i) load_to_lds(rb, vb[i], so, base + kABytes + (wave * kBLoads + i) * 1024);
  };
  const int arow = wm * 64 + (lane & 31), brow = wn * 64 + (lane & 31);
  const uint32_t a_off = (uint32_t)(arow * 128), b_off = (uint32_t)(kABytes + brow * 128);
  const int asw = (arow >> 1) & 7, bsw = (brow >> 1) & 7;
  f32x16_t acc[2][2];
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;
  int issued = 0, fill = 0, slot = 0;
  for (; issued < kStages - 1 && issued < nk; ++issued) issue(issued, fill++);
  for (int s = 0; s < nk; ++s) {
    if (s + 1 < nk) wait_loads<kLoads>();
    else wait_loads<0>();
    __builtin_amdgcn_s_barrier();
    if (issued < nk) {
      issue(issued, fill);
      ++issued;
      fill = fill + 1 == kStages ? 0 : fill + 1;
    }
    const uint32_t st = lds0 + slot * kStage;
#pragma unroll
    for (int kk = 0; kk < kBK; kk += 16) {
      bf16x8_t af[2], bf[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint32_t c = (uint32_t)(kk / 8 + (lane >> 5));
        af[x] = *(BC_LDS bf16x8_t*)(uintptr_t)(st + a_off + x * 32 * 128 + (c ^ asw) * 16);
        bf[x] = *(BC_LDS bf16x8_t*)(uintptr_t)(st + b_off + x * 32 * 128 + (c ^ bsw) * 16);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[x], bf[y], acc[x][y], 0, 0, 0);
    }
    slot = slot + 1 == kStages ? 0 : slot + 1;
  }
  float* o = part + (size_t)z * M * K;
  const int ib = m0 + wm * 64 + 4 * (lane >> 5), jb = k0 + wn * 64 + (lane & 31);
  const bool full = m0 + kBM <= M && k0 + kBN <= K;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int i = ib + x * 32 + 8 * (r >> 2) + (r & 3), j = jb + y * 32;
        if (full || (i < M && j < K)) o[(size_t)i * K + j] = acc[x][y][r];
      }
}

}  // namespace

template <int kWM, int kWN>
static hipError_t fwd_pipe(const void* w, const void* in, float* out, int N, int M, int K, int P, int relu,
                           hipStream_t s) {
  constexpr int kBM = 64 * kWM, kBN = 64 * kWN;
  const int mt = (M + kBM - 1) / kBM, nt = (P + kBN - 1) / kBN, tiles = mt * nt * N;
  constexpr size_t shm = (size_t)kStages * (kBM + kBN) * kBK * 2;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(std::min(tiles, 256)), dim3(64 * kWM * kWN), shm, s, (const uint16_t*)w,
                       (const uint16_t*)in, out, M, K, P, mt, nt, tiles);
    return hipGetLastError();
  };
  return relu ? go(k_mix_fwd_pipe<kWM, kWN, true>) : go(k_mix_fwd_pipe<kWM, kWN, false>);
}

bool mix_fwd_pipe_takes(const void* w, const void* in, int N, int M, int K, int P) {
  if (K % kBK || P % 8 || ((uintptr_t)w & 15) || ((uintptr_t)in & 15)) return false;
  if ((size_t)M * K * 2 >= ((size_t)1 << 31) || (size_t)K * P * 2 >= ((size_t)1 << 31)) return false;
  if (M <= 64) return false;
  const long tiles = M > 128 ? (long)((M + 255) / 256) * ((P + 127) / 128) * N : (long)((P + 255) / 256) * N;
  return tiles >= 192;
}

hipError_t launch_mix_fwd_pipe(const void* w, const void* in, float* out, int N, int M, int K, int P, int relu,
                               hipStream_t s) {
  return M > 128 ? fwd_pipe<4, 2>(w, in, out, N, M, K, P, relu, s) : fwd_pipe<2, 4>(w, in, out, N, M, K, P, relu, s);
}

// Tiles of the weight gradient.
static int wgrad_tiles(int M, int K) { return ((M + 255) / 256) * ((K + 127) / 128); }

bool mix_wgrad_pipe_takes(const void* grad, const void* in, int N, int M, int K, int P) {
  if (P % kBK || ((uintptr_t)grad & 15) || ((uintptr_t)in & 15)) return false;
  if ((size_t)M * P * 2 >= ((size_t)1 << 31) || (size_t)K * P * 2 >= ((size_t)1 << 31)) return false;
  return M > 128 && (long)wgrad_tiles(M, K) * N * (P / kBK) >= 2048;
}

hipError_t launch_mix_wgrad_pipe(const void* grad, const void* in, float* part, int N, int M, int K, int P, int sp,
                                 int chunk, hipStream_t s) {
  const int mt = (M + 255) / 256, nt = (K + 127) / 128, total = mt * nt * N * sp;
  constexpr size_t shm = (size_t)kStages * (256 + 128) * kBK * 2;
  hipLaunchKernelGGL((k_mix_wgrad_pipe<4, 2>), dim3((total + 7) & ~7), dim3(512), shm, s, (const uint16_t*)grad,
                     (const uint16_t*)in, part, M, K, P, mt, nt, sp, chunk, total);
  return hipGetLastError();
}

}  // namespace bc
