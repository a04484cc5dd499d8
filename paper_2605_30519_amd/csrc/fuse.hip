// fuse.hip -- Eq. 1's gated fusion of the three attention branches for gfx950:
//   out[i][h] = sum over c in (CMP, SLC, SWA) of sigmoid(gate[i][h][c]) * o_c[i][h].
// HBM-bound and elementwise: a thread takes 16-byte chunks of one output row, reads the
// row's three gate logits and the matching chunks of each present branch, combines
// in fp32 and stores the chunks rounded to the output dtype.
#include <math.h>

#include "device_common.h"
#include "launch.h"

namespace omnimem {
namespace {

constexpr int kFuseThreads = 256;

// 16 bytes to memory, PAST the caches or as usual.
template <bool PAST>
__device__ __forceinline__ void store16(u32x4 w, void* p) {
  if constexpr (PAST)
    __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
  else
    *reinterpret_cast<u32x4*>(p) = w;
}

template <typename T>
struct Chunk;

template <>
struct Chunk<uint16_t> {
  static constexpr int N = 8;
  template <bool PAST>
  __device__ __forceinline__ static void store(uint16_t* p, const float (&x)[8]) {
    bf16x8 w;  // nearest even, two a conversion
#pragma unroll
    for (int j = 0; j < 8; ++j) w[j] = static_cast<__bf16>(x[j]);
    store16<PAST>(__builtin_bit_cast(u32x4, w), p);
  }
};

template <>
struct Chunk<float> {
  static constexpr int N = 4;
  template <bool PAST>
  __device__ __forceinline__ static void store(float* p, const float (&x)[4]) {
    store16<PAST>(__builtin_bit_cast(u32x4, f32x4{x[0], x[1], x[2], x[3]}), p);
  }
};

// Two chunks of a row per lane, half a row apart (a row's lanes read whole lines where they
// can): the sigmoids, three exponentials and divisions, are formed once for both, and all
// six loads are in flight before the first product.  Bound by its 4 tensors' bytes, from
// HBM or, written just before, from the MALL.  One chunk per lane, the row found by a
// 64-bit division and a branch's loads behind the one before: 4,680 rows x 12 heads, bf16,
// d = 128: 12.0 -> 10.8 us; 8 heads 7.8 -> 6.4; fp32, 1,560 rows 7.0 -> 4.9.  Four chunks
// per lane break the lines (11.0 us).
// The output is stored past the caches, which then hold more of the branches: 40 heads x
// 4,680 rows, fp32 (383 MB) 69.5 -> 54.7 us, 32 heads 48.8 -> 43.9, smaller calls unchanged.
// STREAM reads the branches past the caches instead and stores as usual.  That loses where
// the branches are still there, as after their attention (40 heads, bf16, 192 MB: 28.5 ->
// 32.9 us; the fp32 call of 383 MB 54.7 -> 59.7), and gains where they are more than the
// 256 MB memory-side cache holds for long: 40 heads x 12,000 rows, bf16 (369 MB of branches)
// 87.1 -> 75.9, 9,000 rows, fp32 (553 MB) 129 -> 111.
constexpr int kFuseChunks = 2;
constexpr int64_t kFuseStreamBytes = 320ll << 20;  // bytes of branches

template <typename T, int D>
constexpr int fuse_lanes() {  // lanes per row
  return D / Chunk<T>::N / kFuseChunks;
}

template <typename T, int D, bool STREAM>
__global__ __launch_bounds__(kFuseThreads) void k_gated_combine(const T* __restrict__ o_cmp, const T* __restrict__ o_slc,
                                                                const T* __restrict__ o_swa,
                                                                const float* __restrict__ gate, int64_t rows, T* out) {
  constexpr int N = Chunk<T>::N, LPR = fuse_lanes<T, D>();
  const int64_t row = static_cast<int64_t>(blockIdx.x) * (kFuseThreads / LPR) + threadIdx.x / LPR;
  if (row >= rows) return;
  const int64_t at = row * D + threadIdx.x % LPR * N;  // element offset of the lane's first chunk
  const T* src[3] = {o_cmp, o_slc, o_swa};
  uint4 raw[3][kFuseChunks];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (src[c] == nullptr) continue;
#pragma unroll
    for (int u = 0; u < kFuseChunks; ++u) {
      const T* p = src[c] + at + u * LPR * N;
      raw[c][u] = STREAM ? load_once(p) : *reinterpret_cast<const uint4*>(p);
    }
  }
  float logit[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) logit[c] = gate[row * 3 + c];
  float acc[kFuseChunks][N] = {};
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    if (src[c] == nullptr) continue;
    const float g = 1.0f / (1.0f + expf(-logit[c]));  // the branch's sigmoid gate, in [0, 1]
#pragma unroll
    for (int u = 0; u < kFuseChunks; ++u) {
      float x[N];
      Vec16<T>::widen(raw[c][u], x);
#pragma unroll
      for (int j = 0; j < N; ++j) acc[u][j] = fmaf(g, x[j], acc[u][j]);
    }
  }
#pragma unroll
  for (int u = 0; u < kFuseChunks; ++u) Chunk<T>::template store<!STREAM>(out + at + u * LPR * N, acc[u]);
}

template <typename T, int D>
hipError_t launch_typed(int64_t rows, const void* o_cmp, const void* o_slc, const void* o_swa, const float* gate,
                        void* out, hipStream_t stream) {
  constexpr int per = kFuseThreads / fuse_lanes<T, D>();  // rows per workgroup
  const int64_t blocks = (rows + per - 1) / per;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const int branches = (o_cmp != nullptr) + (o_slc != nullptr) + (o_swa != nullptr);
  const bool stream_in = branches * rows * D * static_cast<int64_t>(sizeof(T)) > kFuseStreamBytes;
  const auto kernel = stream_in ? k_gated_combine<T, D, true> : k_gated_combine<T, D, false>;
  return launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kFuseThreads), 0, stream,
                       static_cast<const T*>(o_cmp), static_cast<const T*>(o_slc), static_cast<const T*>(o_swa), gate,
                       rows, static_cast<T*>(out));
}

}  // namespace

hipError_t launch_gated_combine(int dtype, int64_t rows, int D, const void* o_cmp, const void* o_slc,
                                const void* o_swa, const float* gate, void* out, hipStream_t stream) {
  if (rows <= 0) return hipSuccess;
  if (dtype == 0)
    return D == 128 ? launch_typed<uint16_t, 128>(rows, o_cmp, o_slc, o_swa, gate, out, stream)
                    : launch_typed<uint16_t, 64>(rows, o_cmp, o_slc, o_swa, gate, out, stream);
  return D == 128 ? launch_typed<float, 128>(rows, o_cmp, o_slc, o_swa, gate, out, stream)
                  : launch_typed<float, 64>(rows, o_cmp, o_slc, o_swa, gate, out, stream);
}

}  // namespace omnimem
