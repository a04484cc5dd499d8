// device_common.h -- small device helpers shared by the libomnimem kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace omnimem {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kNumXcd = 8;  // MI355X: 8 accelerator complex dies, workgroups dispatched round-robin

// The hardware dispatches workgroup i to XCD (i mod 8).  Remap so that the
// workgroups that land on one XCD get a contiguous range of logical ids; work that
// shares data (all query tiles of one head) then shares that XCD's L2.
__device__ __forceinline__ int xcd_contiguous_id(int bid, int nblocks) {
  const int per = nblocks / kNumXcd, rem = nblocks % kNumXcd;
  const int xcd = bid % kNumXcd, local = bid / kNumXcd;
  return xcd < rem ? xcd * (per + 1) + local : rem * (per + 1) + (xcd - rem) * per + local;
}

// 16-byte load with the nontemporal hint, for data read once (the K stream of the
// selection, Q): it is not kept in the caches, and on gfx950 a stream of such loads
// sustains ~6.3 TB/s against ~5.6 TB/s for plain loads.
__device__ __forceinline__ uint4 load_once(const void* p) {
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}

__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// fp32 -> bf16 bit pattern, rounded to nearest even (NaN stays a quiet NaN).
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x) {
  const uint32_t u = __float_as_uint(x);
  if ((u & 0x7fffffffu) > 0x7f800000u) return static_cast<uint16_t>((u >> 16) | 0x40u);
  return static_cast<uint16_t>((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Order-preserving map of an fp32 score to uint32 (larger score -> larger key).
// -0 is folded onto +0 first so that equal scores compare equal.  Candidate keys
// are forced >= 1 so that 0 can mark "not a candidate".
__device__ __forceinline__ uint32_t score_key(float s) {
  s = s + 0.0f;
  const uint32_t u = __float_as_uint(s);
  const uint32_t k = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return k == 0u ? 1u : k;
}

// ---------------------------------------------------------------- tiles in LDS by DMA
constexpr int kTileKeys = 64;  // keys per tile (one B = 64 block, half of a B = 128 block, one compressed page)

// LDS tiles of 64 keys for the MFMA kernels: rows of 2 d bytes, unpadded, with the 16-byte
// chunks of each row permuted so that both the K fragment reads (one chunk of 16 rows a
// pass) and the transposing V reads (4 chunks of 4 rows a pass) touch every bank once:
//   K: chunk c of row r sits at chunk position c ^ (r mod 16), for d = 64, where two rows
//      span the banks, at c ^ (r / 2 mod 8)
//   V: at c ^ 4 (r mod 4), for d = 64 at c ^ 4 (r / 2 mod 2)
// Tiles arrive by buffer-to-LDS DMA: one instruction moves 64 lanes x 16 bytes into a
// contiguous 1 KB (4 rows, for d = 64 8), lane l filling position l mod (d / 8) of its
// row, so each lane fetches the global chunk that belongs at its position.
template <int D>
struct KeyTileLds {
  static constexpr int ROW = D * 2;                 // bytes per row
  static constexpr int TILE = kTileKeys * ROW;      // bytes per tile
  static constexpr int CHUNKS = D / 8;              // 16-byte chunks per row
  static constexpr int DMA_ROWS = 1024 / ROW;       // rows per DMA instruction
  __device__ __forceinline__ static int k_pos(int r, int c) {
    return r * ROW + ((c ^ (D == 128 ? r & 15 : (r >> 1) & 7)) << 4);
  }
  __device__ __forceinline__ static int v_pos(int r, int c) {
    return r * ROW + ((c ^ (D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1))) << 4);
  }
};

// Workgroup barrier for LDS traffic only.  __syncthreads() also orders global memory,
// which makes every wave drain its outstanding loads, including the DMA of tiles
// meant to stay in flight across the barrier; LDS written by DMA is covered by the
// explicit vmcnt wait before it, and the asm statements keep the compiler from
// moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt operand that waits for at most n outstanding vector-memory operations
// and for nothing else (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
constexpr int vmcnt_only(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }

// Buffer resource (raw, stride 0) over `bytes` bytes at p, in scalar registers; the
// caller guarantees p and bytes are the same in every lane.  Offsets at or past the
// end read as zero.
__device__ __forceinline__ u32x4 buffer_rsrc(const void* p, int bytes) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  u32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u));
  r[1] = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(u >> 32) & 0xffffu);
  r[2] = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(bytes));
  r[3] = 0x00020000u;
  return r;
}

__device__ __forceinline__ uint32_t lds_offset(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) const void*)p));
}

// One buffer-to-LDS DMA instruction: lane l's 16 bytes at rsrc + voffset land at LDS
// byte lds + 16 l.  It is written as inline asm so that the compiler does not track
// it as an LDS store (it would make every later LDS read wait for all DMA in flight);
// the kernel orders it itself, with explicit vmcnt waits before the barriers that
// publish a stage.
__device__ __forceinline__ void dma_16x64(u32x4 rsrc, int voffset, uint32_t lds) {
  // M0 (the LDS destination) is set by the compiler; the s_nop is the wait state an
  // LDS DMA needs after an M0 write
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds" ::"v"(voffset), "s"(rsrc), "{m0}"(lds) : "memory");
}

// 16-byte vector load widened to fp32: 8 bf16 or 4 fp32 values.
template <typename T>
struct Vec16;

template <>
struct Vec16<uint16_t> {  // bf16 storage
  static constexpr int N = 8;
  __device__ __forceinline__ static void load(const uint16_t* p, float (&out)[8]) {
    widen(*reinterpret_cast<const uint4*>(p), out);
  }
  __device__ __forceinline__ static void widen(const uint4 raw, float (&out)[8]) {
    const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      out[2 * i] = __uint_as_float(w[i] << 16);
      out[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

template <>
struct Vec16<float> {
  static constexpr int N = 4;
  __device__ __forceinline__ static void load(const float* p, float (&out)[4]) {
    widen(*reinterpret_cast<const uint4*>(p), out);
  }
  __device__ __forceinline__ static void widen(const uint4 raw, float (&out)[4]) {
    out[0] = __uint_as_float(raw.x);
    out[1] = __uint_as_float(raw.y);
    out[2] = __uint_as_float(raw.z);
    out[3] = __uint_as_float(raw.w);
  }
};

__device__ __forceinline__ float wave_xor_sum(float v, int lane_mask_lo, int lane_mask_hi) {
  for (int m = lane_mask_lo; m <= lane_mask_hi; m <<= 1) v += __shfl_xor(v, m);
  return v;
}

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  const int lane = threadIdx.x % kWave;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int t = __shfl_up(v, off);
    if (lane >= off) v += t;
  }
  return v;
}

// Exclusive prefix sum over a workgroup of NT threads; `total` gets the sum.
// `tmp` must hold NT/64 ints of LDS.  Contains barriers: call from all threads.
template <int NT>
__device__ __forceinline__ int block_exclusive_scan(int v, int* tmp, int& total) {
  constexpr int kWaves = NT / kWave;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int incl = wave_inclusive_scan(v);
  if (lane == kWave - 1) tmp[wave] = incl;
  __syncthreads();
  int before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const int t = tmp[w];
    if (w < wave) before += t;
    sum += t;
  }
  __syncthreads();
  total = sum;
  return before + incl - v;
}

}  // namespace omnimem
