// attention.hip -- attention over per-(head, group) block lists read in place from
// the paged KV cache (Sec. 3.3 Eq. 5, Per-Head Scattered KV Access; App. C Alg. 1
// Step 2), and over contiguous chunk ranges (dense / sliding-window attention).
//
// bf16 kernels: flash-style, a group's block list walked 64 keys at a time (one
// (page, head) slab, or half of one at B = 128).  A wave keeps 32-row tiles of Q in
// registers and computes, for each,
//   S^T = K Q^T        on v_mfma_f32_32x32x16_bf16 (K rows as the A operand),
//   O^T += V^T P^T     on the same instruction, V^T read with ds_read_b64_tr_b16,
// so that each lane owns one query column of both S^T and O^T: the online softmax
// (fp32, exp2 domain with the scale folded in) and the rescaling of O need one
// cross-lane exchange (lane l <-> l^32) per tile and no transposes.  The A-operand
// rows of K are fed in an order (bits 2 and 3 of the row swapped) that makes the
// S^T accumulator registers line up with the B-operand layout of P^T, so P goes from
// accumulator to MFMA operand with a bf16 pack and nothing else.
//
// The same formulation runs in three shapes: k_attn_bf16_r64 (d = 128, groups of more than
// 32 rows: 64 rows per wave) and k_attn_bf16_r32 (d = 64, the same groups: 32 rows per wave),
// both with tiles by buffer-to-LDS DMA and the keys split over sets of waves where the grid
// is small; and k_attn_bf16_groups (groups of at most 32 rows: one wave per group, every
// wave streaming its own groups' tiles).
//
// f32 kernel (k_attn_f32): the same formulation on fp32 MFMA, the keys of a 32-row tile
// split over the waves of its workgroup, for fp32 inputs.
#include <limits.h>
#include <math.h>
#include <atomic>
#include <type_traits>

#include "device_common.h"
#include "launch.h"

namespace omnimem {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

struct AttnArgs {
  const void* q;
  const void* k_pages;
  const void* v_pages;
  const int32_t* page_table;
  int64_t pt_stride;  // 0: one table for every head; else head h's table at h * pt_stride
  int64_t num_pages;
  int H, S, B, Bpc, nb;
  int lq, G, R;
  const int32_t* idx;
  const int32_t* cnt;
  int top_k;
  int dense_first, dense_count;
  float scale;
  void* out;
  float* lse;
  int tiles_per_group;
  int first_wg;  // workgroups of the call before this grid
};

__device__ __forceinline__ void resolve_tile(const AttnArgs& a, int id, int rows_per_wg, int& h, int& hr, int& row0,
                                             int& row_end) {
  const int tile = id % a.tiles_per_group;
  hr = id / a.tiles_per_group;
  const int r = hr % a.R;
  h = hr / a.R;
  const int g_begin = r * a.G;
  const int g_end = min(g_begin + a.G, a.lq);
  row0 = g_begin + tile * rows_per_wg;
  row_end = min(row0 + rows_per_wg, g_end);
}

// The page table head h reads.
__device__ __forceinline__ const int32_t* head_table(const AttnArgs& a, int h) {
  return a.page_table + static_cast<int64_t>(h) * a.pt_stride;
}

__device__ __forceinline__ void resolve_list(const AttnArgs& a, int hr, const int32_t*& list, int& count) {
  if (a.idx) {
    list = a.idx + static_cast<int64_t>(hr) * a.top_k;
    const int c = a.cnt[hr];
    count = c < 0 ? 0 : (c > a.top_k ? a.top_k : c);
  } else {
    list = nullptr;
    count = a.dense_count;
  }
}

// Decodes list entries [first, first + NT) into a compact table of 64-key tiles in
// LDS: entry i = (page, (sub-tile << 8) | valid keys).  Padding, out-of-range ids and
// non-resident pages produce no tile; a B = 128 block produces up to two.  One list
// entry per thread, compacted with a block-wide prefix sum; returns the tile count.
// Contains barriers: every thread of the workgroup must call it.  pre_id, unless
// INT_MIN, is this thread's list entry, already read by the caller.
template <int NT>
__device__ int decode_tiles(const AttnArgs& a, const int32_t* pt, const int32_t* list, int count, int first,
                            int2* table, int* scan_tmp, int pre_id = INT_MIN) {
  const int e = first + static_cast<int>(threadIdx.x);
  int ntiles = 0, page = 0, nvb = 0;
  if (e < count) {
    const int id = pre_id != INT_MIN ? pre_id : list ? list[e] : a.dense_first + e;
    if (id >= 0 && id < a.nb) {
      const int32_t p = pt[id];
      if (p >= 0 && p < a.num_pages) {
        const int o = id % a.Bpc;
        nvb = o == a.Bpc - 1 ? a.S - o * a.B : a.B;
        page = p;
        ntiles = (nvb + kTileKeys - 1) / kTileKeys;
      }
    }
  }
  int total;
  const int pos = block_exclusive_scan<NT>(ntiles, scan_tmp, total);
  for (int s = 0; s < ntiles; ++s) {
    const int nv = nvb - s * kTileKeys;
    table[pos + s] = make_int2(page, (s << 8) | (nv < kTileKeys ? nv : kTileKeys));
  }
  __syncthreads();
  return total;
}

// ------------------------------------------------------------------ bf16 / MFMA
// A-operand row order for S^T = K Q^T: swapping bits 2 and 3 of the row makes the
// accumulator element i of lane l hold key 8*(l/32)+i (i < 8) or 16+8*(l/32)+(i-8).
__device__ __forceinline__ int s_row_perm(int x) { return (x & ~12) | ((x & 4) << 1) | ((x & 8) >> 1); }

// LDS row stride of a V tile (bf16 elements), chosen for gfx950's 64 four-byte banks: V
// rows are read by ds_read_b64_tr_b16, 4 rows x 32 B per 16-lane group and two groups per
// pass: a stride of 16 or 48 (mod 64) dwords makes the 8 row segments of a pass disjoint.
template <int D>
struct AttnLds {
  static constexpr int V_STRIDE = D == 128 ? 160 : 96;
  static constexpr int V_ELEMS = kTileKeys * V_STRIDE;
};

// ------------------------------------------------------------------ bf16 / MFMA, one wave per query group
// Query groups of at most 32 rows (the small-group setting of App. B, where every
// group of G_q rows keeps its own top-K blocks, and short dense calls): a group is
// one 32-row MFMA tile, so its attention is a gather with little arithmetic per
// byte.  Every wave runs on its own, with no barrier: it walks a sequence of
// (head, group) pairs (pair first + k * stride, the grid resident at once), and
// the tiles of consecutive groups form one stream, the next tile's K and V always
// in flight while the current one is computed, across group boundaries too.  K
// goes from memory straight into registers in the MFMA A-operand layout; V passes
// through the wave's own LDS tile for the transposing reads.  Lists are read two groups
// ahead and their pages one, a group's Q rows with its first tile.
// Operand layouts and rounding are those of the kernels for larger groups; the online
// softmax is the plain one of k_attn_bf16_r32 (the true running max).
// Bound by the gathers where groups fill the waves (12 heads x 312 groups x 4 blocks:
// 520 MB at 6.0 TB/s), by one wave's chain of loads and a tile's work where they do not.
// With a count, list and table read in series before a group's first tile, and each load
// of 16 bytes a branch on its row with its register cleared first, those took 88.8 us and,
// 3 heads x 104 groups (a wave each), 21.9; now 87.1 and 17.4; groups of 32 rows, 40 heads,
// 8 blocks 88.5 -> 84.8.  K by whole rows through LDS instead: 102 us, the tile's work then
// waits for two more trips through LDS.
constexpr int kGrpWaves = 4;

template <int D>
__global__ __launch_bounds__(kGrpWaves* kWave, 1) void k_attn_bf16_groups(AttnArgs a) {
  using L = AttnLds<D>;
  constexpr int KK = D / 16;                       // k-steps of QK^T
  constexpr int DT = D / 32;                       // 32-wide output tiles along d
  constexpr int CPR = D / 8;                       // 16-byte chunks per key row
  constexpr int VROWS = kWave / CPR;               // V rows per load instruction
  constexpr int VLOADS = kTileKeys / VROWS;        // V load instructions per tile
  __shared__ __attribute__((aligned(16))) uint16_t v_all[kGrpWaves * L::V_ELEMS];

  const int lane = threadIdx.x % kWave, half = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  uint16_t* const v_lds = v_all + wave * L::V_ELEMS;
  const int total = a.H * a.R;
  const int stride = gridDim.x * kGrpWaves;
  const int first = xcd_contiguous_id(blockIdx.x, gridDim.x) * kGrpWaves + wave;
  if (first >= total) return;  // wave-uniform; no barrier anywhere below
  const uint16_t* qp = static_cast<const uint16_t*>(a.q);
  const uint16_t* kp = static_cast<const uint16_t*>(a.k_pages);
  const uint16_t* vp = static_cast<const uint16_t*>(a.v_pages);
  uint16_t* op = static_cast<uint16_t*>(a.out);
  const float c = a.scale * kLog2e;
  const int krow = s_row_perm(lane % 32);

  // ---- the walk over groups and tiles (wave-uniform state; w_*, nx_* and far_id per lane).
  // The lists are read ahead: on entering a group, the next group's pages (nx_page) and the
  // ids and count of the one after (far_*) are asked for and not waited for, so that no
  // chain of list and table reads stands before a group's first tile.
  int p_hr = first, p_count = 0, p_base = 0, p_e = 0, p_sub = 0, p_emitted = 0;
  int w_page = -1, w_nvb = 0;  // entry p_base + lane: page (-1: no tile) and valid tokens
  int nx_id = -1, nx_count = 0, nx_page = -1, far_id = -1, far_count = 0;

  // entry `lane` of a group's list, and its count, as memory has them (an entry past the
  // count is read, never used)
  auto fetch_ids = [&](int hr, int& id, int& count) {
    id = -1;
    count = 0;
    if (hr >= total) return;
    count = a.dense_count;
    if (a.idx) {
      count = a.cnt[hr];
      if (lane < a.top_k) id = a.idx[static_cast<int64_t>(hr) * a.top_k + lane];
    } else {
      id = a.dense_first + lane;
    }
  };
  auto fetch_page = [&](int hr, int id) -> int { return id >= 0 && id < a.nb ? head_table(a, hr / a.R)[id] : -1; };
  // this lane's entry of the window: its page and valid tokens, or no tile
  auto set_window = [&](int e, int id, int p) {
    w_page = -1;
    w_nvb = 0;
    if (e < p_count && id >= 0 && id < a.nb) {
      const int o = id % a.Bpc;
      const int nvb = o == a.Bpc - 1 ? a.S - o * a.B : a.B;
      if (p >= 0 && p < a.num_pages && nvb > 0) {
        w_page = p;
        w_nvb = nvb;
      }
    }
  };
  // enters group p_hr, whose entries are in nx_*
  auto enter_group = [&]() {
    const int most = a.idx ? a.top_k : a.dense_count;
    p_count = __builtin_amdgcn_readfirstlane(min(max(nx_count, 0), most));
    p_base = p_e = p_sub = p_emitted = 0;
    set_window(lane, nx_id, nx_page);
    nx_id = far_id;
    nx_count = far_count;
    nx_page = fetch_page(p_hr + stride, nx_id);
    fetch_ids(p_hr + 2 * stride, far_id, far_count);
  };
  // output of a group without a single tile: O = 0, lse = -inf
  auto write_empty = [&](int hr) {
    const int h = hr / a.R, g0 = (hr % a.R) * a.G, rows = min(g0 + a.G, a.lq) - g0;
    for (int i = lane; i < rows * CPR; i += kWave)
      *reinterpret_cast<uint4*>(op + (static_cast<int64_t>(g0 + i / CPR) * a.H + h) * D + (i % CPR) * 8) =
          make_uint4(0, 0, 0, 0);
    if (a.lse && lane < rows) a.lse[static_cast<int64_t>(h) * a.lq + g0 + lane] = -INFINITY;
  };
  fetch_ids(first, nx_id, nx_count);
  fetch_ids(first + stride, far_id, far_count);
  nx_page = fetch_page(first, nx_id);
  enter_group();

  // the next tile of the walk: page, (sub-tile << 8) | valid keys, its group, and
  // whether it opens the group; false at the end
  auto next_tile = [&](int& page, int& meta, int& hr, bool& opens) -> bool {
    for (;;) {
      while (p_e < p_count) {
        if (p_e >= p_base + kWave) {  // lists longer than a wave: the next window
          p_base += kWave;
          const int e = p_base + lane;
          int id = -1;
          if (e < p_count) id = a.idx ? a.idx[static_cast<int64_t>(p_hr) * a.top_k + e] : a.dense_first + e;
          set_window(e, id, fetch_page(p_hr, id));
          continue;
        }
        const uint64_t live = __ballot(w_page >= 0) & (~0ull << (p_e - p_base));
        if (live == 0) {
          p_e = p_base + kWave;
          p_sub = 0;
          continue;
        }
        const int l = __builtin_ctzll(live);
        if (p_base + l != p_e) {
          p_e = p_base + l;
          p_sub = 0;
        }
        const int nvb = __builtin_amdgcn_readlane(w_nvb, l);
        page = __builtin_amdgcn_readlane(w_page, l);
        const int left = nvb - p_sub * kTileKeys;
        meta = (p_sub << 8) | (left < kTileKeys ? left : kTileKeys);
        hr = p_hr;
        opens = p_emitted == 0;
        ++p_emitted;
        if (++p_sub * kTileKeys >= nvb) {
          ++p_e;
          p_sub = 0;
        }
        return true;
      }
      if (p_emitted == 0) write_empty(p_hr);
      p_hr += stride;
      if (p_hr >= total) return false;
      enter_group();
    }
  };

  // ---- registers of the stream: K of two tiles (current, next), V of the next, Q
  bf16x8 ka[2][KK], kb[2][KK], q[KK], qn[KK];
  uint4 vn[VLOADS];
  // Read through buffer descriptors that end at the last valid key: rows past it read as
  // zero, with no branch around a load and no register to clear before it.
  auto tile_rsrc = [](const uint16_t* p, int bytes) {
    const u32x4 r = buffer_rsrc(p, bytes);
    return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(static_cast<uint64_t>(r[1]) << 32 | r[0]), 0, r[2], r[3]);
  };
  auto load_tile = [&](int page, int meta, int hr, bf16x8 (&kf)[2][KK]) {
    const int sub = meta >> 8, nv = meta & 255;
    const int64_t slab = (static_cast<int64_t>(page) * a.H + hr / a.R) * a.B * D + static_cast<int64_t>(sub) * kTileKeys * D;
    const auto ks = tile_rsrc(kp + slab, nv * D * 2), vs = tile_rsrc(vp + slab, nv * D * 2);
    const int at = krow * D * 2 + 16 * half;
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
        kf[t2][kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ks, at + 32 * kk, 32 * t2 * D * 2, 0));
#pragma unroll
    for (int i = 0; i < VLOADS; ++i)
      vn[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(vs, lane * 16 + i % 4 * 1024, i / 4 * 4096, 0));
  };
  auto load_q = [&](int hr) {
    const int h = hr / a.R, g0 = (hr % a.R) * a.G, g1 = min(g0 + a.G, a.lq);
    // rows past the group's last one repeat it: their results are not stored
    const uint16_t* row = qp + (static_cast<int64_t>(min(g0 + lane % 32, g1 - 1)) * a.H + h) * D + 8 * half;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qn[kk] = *reinterpret_cast<const bf16x8*>(row + 16 * kk);
  };

  // ---- per-group softmax state
  f32x16 o_acc[DT];
  float m_run = -INFINITY, l_run = 0.f;
  int cur_hr = -1;
  auto finish = [&](int hr) {
    const int h = hr / a.R, g0 = (hr % a.R) * a.G, g1 = min(g0 + a.G, a.lq);
    const int row = g0 + lane % 32;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
    if (row < g1) {
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          bf16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(o_acc[dt][4 * i4 + e] * inv);
          *reinterpret_cast<bf16x4*>(op + (static_cast<int64_t>(row) * a.H + h) * D + 32 * dt + 8 * i4 + 4 * half) = w;
        }
      if (a.lse && lane < 32)
        a.lse[static_cast<int64_t>(h) * a.lq + row] = l_tot > 0.f ? (m_run * c + __log2f(l_tot)) * kLn2 : -INFINITY;
    }
  };
  auto open_group = [&](int hr) {
    if (cur_hr >= 0) finish(cur_hr);
    cur_hr = hr;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) q[kk] = qn[kk];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o_acc[dt][i] = 0.f;
    m_run = -INFINITY;
    l_run = 0.f;
  };

  bf16x8 pb[4];
  auto pv = [&]() {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int key0 = 16 * j + 8 * half + (lane % 16) / 4;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int col = 32 * dt + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
        typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(v_lds + key0 * L::V_STRIDE + col));
        const i16x4 hi =
            __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(v_lds + (key0 + 4) * L::V_STRIDE + col));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o_acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pb[j], o_acc[dt], 0, 0, 0);
      }
    }
  };
  // QK^T, online softmax and PV of one tile whose K is in kf and V in the LDS tile
  auto compute = [&](const bf16x8 (&kf)[2][KK], int nvalid) {
    f32x16 s_acc[2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2) {
#pragma unroll
      for (int i = 0; i < 16; ++i) s_acc[t2][i] = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) s_acc[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[t2][kk], q[kk], s_acc[t2], 0, 0, 0);
    }
    if (nvalid < kTileKeys) {  // partial tile: mask the keys past the block's end
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = 32 * t2 + (i < 8 ? 8 * half + i : 16 + 8 * half + (i - 8));
          if (key >= nvalid) s_acc[t2][i] = -INFINITY;
        }
    }
    float mloc = s_acc[0][0];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 16; ++i) mloc = fmaxf(mloc, s_acc[t2][i]);
    const float m_tile = fmaxf(mloc, __shfl_xor(mloc, 32));
    if (__any(m_tile > m_run)) {  // rescale only when some lane's running max grows
      const float m_new = fmaxf(m_run, m_tile);
      const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * c);
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) o_acc[dt][i] *= alpha;
      m_run = m_new;
    }
    const float mc = m_run == -INFINITY ? 0.f : m_run * c;
    float psum = 0.f;
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s_acc[t2][i], c, -mc));
        psum += p;
        pb[2 * t2 + i / 8][i % 8] = static_cast<__bf16>(p);
      }
    l_run += psum;
    pv();
  };

  int page = 0, meta = 0, hr = 0;
  bool opens = false;
  bool have = next_tile(page, meta, hr, opens);
  if (have) {
    load_tile(page, meta, hr, ka);
    if (opens) load_q(hr);
  }
  // one tile: its K in kc, its V in vn; the next tile's loads go to kn and vn
  auto step = [&](bf16x8 (&kc)[2][KK], bf16x8 (&kn)[2][KK]) {
    const int nvalid = meta & 255;
    if (opens) open_group(hr);
#pragma unroll
    for (int i = 0; i < VLOADS; ++i)
      *reinterpret_cast<uint4*>(v_lds + (i * VROWS + lane / CPR) * L::V_STRIDE + (lane % CPR) * 8) = vn[i];
    have = next_tile(page, meta, hr, opens);
    if (have) {
      load_tile(page, meta, hr, kn);
      if (opens) load_q(hr);
    }
    compute(kc, nvalid);
  };
  while (have) {
    step(ka, kb);
    if (!have) break;
    step(kb, ka);
  }
  if (cur_hr >= 0) finish(cur_hr);
}

// max / sum of a value over the lane pair (l, l ^ 32)
__device__ __forceinline__ float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ------------------------------------------------------------------ bf16 / MFMA, 32 rows per wave
// d = 64, groups of more than 32 rows: 8 waves, two per SIMD, each own 32 query rows, and the
// two of a SIMD run a tile half a step apart: waves 0-3 do QK(t), softmax(t), PV(t); waves
// 4-7 PV(t-1), QK(t), softmax(t), so that one issues MFMAs while the other is in its softmax.
// The softmax bounds it: of a SIMD's cycles VALU work issues for 64% (some 200 operations a
// wave and tile, 33 of them exponentials), the MFMA pipe is busy for 32%, half of that under
// the VALU work, and a fifth has neither.
// The max of a row is the true one of the tiles so far, so a row's largest P is 1 and its
// bf16 exact.  A max that lags, as the 64-row kernel's does, rounds the largest P like any
// other: outputs 2.33e-3 off fp64 against 2.21e-3 (16 heads x 1,560 rows x 4,680 keys).
// KS key streams: the waves are KS sets of 8 / KS, set j taking tiles j, j + KS, ... of the
// list; they meet in LDS at the end.  K and V tiles arrive by DMA, a tile ahead, in two
// stages; where one stream's waves run half a step apart (KS = 1), V has three.
// 16 heads x 1,560 rows x 64 tiles, two streams: 43.5 us (replayed from a graph), as the
// 64-row scheme at d = 64 took (43.6); tiles through registers, one stream, 93.2.
constexpr int kR32Waves = 8;

template <int KS>
__global__ __launch_bounds__(kR32Waves* kWave) void k_attn_bf16_r32(AttnArgs a) {
  constexpr int D = 64;
  using L = KeyTileLds<D>;
  constexpr int NT = kR32Waves * kWave;
  constexpr int RW = kR32Waves / KS;  // row waves per stream
  constexpr int ROWS = RW * 32;
  constexpr int DT = D / 32;
  constexpr int KK = D / 16;
  constexpr int DMA_PER_WAVE = L::TILE / 1024 / RW;
  constexpr int V_STAGES = KS == 1 ? 3 : 2;
  constexpr int kKBytes = KS * 2 * L::TILE, kVBytes = KS * V_STAGES * L::TILE;
  __shared__ __attribute__((aligned(1024))) uint8_t lds[kKBytes + kVBytes];
  __shared__ __attribute__((aligned(16))) int2 table[2 * NT];
  __shared__ int scan_tmp[kR32Waves];

  int h, hr, row0, row_end;
  resolve_tile(a, xcd_contiguous_id(blockIdx.x, gridDim.x), ROWS, h, hr, row0, row_end);
  if (row0 >= row_end) return;  // workgroup-uniform: no barrier has been reached
  const int32_t* list;
  int count;
  resolve_list(a, hr, list, count);

  const int tid = threadIdx.x, lane = tid % kWave, half = lane / 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wave_r = wave % RW, stream = wave / RW;
  const bool late = wave >= kR32Waves / 2;
  // this thread's entry of the first decoded stretch, read without waiting for the count
  const int id0 = list != nullptr && tid < a.top_k ? list[tid] : INT_MIN;
  const uint16_t* qp = static_cast<const uint16_t*>(a.q);
  const float c = a.scale * kLog2e;

  // Q^T as the B operand: lane holds query wrow + lane % 32, d = 16 kk + 8 half + 0..7
  const int wrow = row0 + wave_r * 32;
  const bool wave_live = wrow < row_end;  // wave-uniform
  bf16x8 q[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    q[kk] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    if (wrow + lane % 32 < row_end)
      q[kk] = *reinterpret_cast<const bf16x8*>(qp + (static_cast<int64_t>(wrow + lane % 32) * a.H + h) * D + 16 * kk + 8 * half);
  }
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;  // running max (raw score units), this lane's share of l

  // ---- tile sequence: (page, sub-tile << 8 | valid keys); every stream takes its own of the
  // next KS entries (an empty tile past the table's end), `more` tells whether there was one
  // for any of them.  Called by every thread together: it refills the table (with barriers).
  int next_entry = 0, ntab = 0, ti = 0;
  bool more = false;
  auto next_tile = [&]() -> int2 {
    if (ti >= ntab) {
      ntab = 0;
      ti = 0;
      while (ntab == 0 && next_entry < count) {
        ntab = decode_tiles<NT>(a, head_table(a, h), list, count, next_entry, table, scan_tmp,
                                next_entry == 0 ? id0 : INT_MIN);
        next_entry += NT;
      }
      ntab = __builtin_amdgcn_readfirstlane(ntab);
    }
    more = ti < ntab;
    const int2 m = ti + stream < ntab ? table[ti + stream] : make_int2(0, 0);
    ti += KS;
    return make_int2(__builtin_amdgcn_readfirstlane(m.x), __builtin_amdgcn_readfirstlane(m.y));
  };

  // ---- DMA of the wave's share of a tile (instructions wave_r + RW i); an empty tile loads
  // nothing and writes zeros, rows past the last valid key read as zero
  const int64_t h_elems = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(h)) * a.B * D;
  const int64_t page_elems = static_cast<int64_t>(a.H) * a.B * D;
  const uint16_t* const kp_h = static_cast<const uint16_t*>(a.k_pages) + h_elems;
  const uint16_t* const vp_h = static_cast<const uint16_t*>(a.v_pages) + h_elems;
  uint8_t* const k_ring = lds + stream * 2 * L::TILE;
  uint8_t* const v_ring = lds + kKBytes + stream * V_STAGES * L::TILE;
  const uint32_t k_dst = lds_offset(k_ring) + wave_r * 1024, v_dst = lds_offset(v_ring) + wave_r * 1024;
  int k_src[DMA_PER_WAVE], v_src[DMA_PER_WAVE];
#pragma unroll
  for (int i = 0; i < DMA_PER_WAVE; ++i) {
    const int r = L::DMA_ROWS * (wave_r + RW * i) + lane / L::CHUNKS, p = lane % L::CHUNKS;
    k_src[i] = L::k_pos(r, p);
    v_src[i] = L::v_pos(r, p);
  }
  auto rsrc_of = [&](const uint16_t* base, int2 m) {
    return buffer_rsrc(base + m.x * page_elems + static_cast<int64_t>(m.y >> 8) * kTileKeys * D, (m.y & 255) * L::ROW);
  };
  auto issue_k = [&](int2 m, int st) {
    const u32x4 r = rsrc_of(kp_h, m);
#pragma unroll
    for (int i = 0; i < DMA_PER_WAVE; ++i) dma_16x64(r, k_src[i], k_dst + st * L::TILE + RW * i * 1024);
  };
  auto issue_v = [&](int2 m, int st) {
    const u32x4 r = rsrc_of(vp_h, m);
#pragma unroll
    for (int i = 0; i < DMA_PER_WAVE; ++i) dma_16x64(r, v_src[i], v_dst + st * L::TILE + RW * i * 1024);
  };
  // this wave's LDS reads have returned and its DMA has landed, and every wave's
  auto step_barrier = [&]() {
    __builtin_amdgcn_s_waitcnt(0x70);  // vmcnt 0, lgkmcnt 0
    lds_barrier();
  };

  const int krow = s_row_perm(lane % 32);
  const int v_key = 8 * half + (lane % 16) / 4, v_chunk = 2 * ((lane / 16) % 2) + (lane % 4) / 2;
  bf16x8 pb[4];
  auto pv = [&](int st) {
    typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        uint8_t* p = v_ring + st * L::TILE + L::v_pos(v_key, 4 * dt + v_chunk) + 8 * (lane % 2) + 16 * j * L::ROW;
        const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
        const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * L::ROW));
        const bf16x8 vf = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pb[j], o[dt], 0, 0, 0);
      }
  };
  // scores and softmax of the tile whose K is in stage st
  auto scores = [&](int st, int nvalid) {
    f32x16 s[2];
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 k = *reinterpret_cast<const bf16x8*>(k_ring + st * L::TILE + L::k_pos(krow, 2 * kk + half) + 32 * t2 * L::ROW);
        s[t2] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q[kk], kk ? s[t2] : f32x16{}, 0, 0, 0);
      }
    if (__builtin_expect(nvalid < kTileKeys, 0)) {  // partial tile: mask the keys past the block's end
      int kb = 8 * half;
      asm volatile("" : "+v"(kb));  // a branch, not 32 selects in every tile
#pragma unroll
      for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = 32 * t2 + (i < 8 ? kb + i : 16 + kb + (i - 8));
          if (key >= nvalid) s[t2][i] = -INFINITY;
        }
    }
    float m0 = fmaxf(s[0][0], s[1][0]), m1 = fmaxf(s[0][1], s[1][1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) {
      m0 = fmaxf(m0, fmaxf(s[0][i], s[1][i]));
      m1 = fmaxf(m1, fmaxf(s[0][i + 1], s[1][i + 1]));
    }
    // rescaled in every tile: some of 32 rows' max grows in most, and a branch around the
    // products costs as many register copies
    const float m_new = fmaxf(m_run, pair_max(fmaxf(m0, m1)));
    const float base = m_new == -INFINITY ? 0.f : m_new, mc = base * c;
    const float alpha = __builtin_amdgcn_exp2f((m_run - base) * c);
    m_run = m_new;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
    float sum[2] = {0.f, 0.f};
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float p = __builtin_amdgcn_exp2f(fmaf(s[t2][i], c, -mc));
        sum[i % 2] += p;
        pb[2 * t2 + i / 8][i % 8] = static_cast<__bf16>(p);
      }
    l_run = fmaf(l_run, alpha, sum[0] + sum[1]);
  };

  // ---- Step t uses K(t) and V(t) (late waves V(t-1)) while K(t+1) and V(t+1) arrive; a
  // stream of late waves takes V a step later, so that two stages hold it.  "V(-1)" is an
  // empty tile's zeros, and P is zero before the first tile.
  const bool v_later = KS > 1 && late;
  int2 cur = next_tile();
  bool cur_more = more;
  issue_v(make_int2(0, 0), V_STAGES - 1);
#pragma unroll
  for (int j = 0; j < 4; ++j) pb[j] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  if (cur_more) {
    issue_k(cur, 0);
    if (!v_later) issue_v(cur, 0);
  }
  step_barrier();
  // One loop for each kind of wave (all of them meet at the same barriers): a branch around
  // the products inside the loop would copy their accumulators.
  auto walk = [&](auto live_, auto late_) {
    constexpr bool LIVE = decltype(live_)::value, LATE = decltype(late_)::value;
    int vst = 0, vprev = V_STAGES - 1;  // V(t)'s stage, V(t-1)'s
    for (int t = 0; cur_more; ++t) {
      const int2 nxt = next_tile();
      const bool nxt_more = more;
      const int vnext = vst + 1 == V_STAGES ? 0 : vst + 1;
      if (nxt_more) issue_k(nxt, (t + 1) % 2);
      if (v_later)
        issue_v(cur, vst);
      else if (nxt_more)
        issue_v(nxt, vnext);
      if constexpr (LIVE) {
        if constexpr (LATE) pv(vprev);
        scores(t % 2, cur.y & 255);
        if constexpr (!LATE) pv(vst);
      }
      step_barrier();
      vprev = vst;
      vst = vnext;
      cur = nxt;
      cur_more = nxt_more;
    }
    if constexpr (LIVE && LATE) pv(vprev);  // the last tile's
  };
  if (!wave_live)
    walk(std::false_type{}, std::false_type{});
  else if (late)
    walk(std::true_type{}, std::true_type{});
  else
    walk(std::true_type{}, std::false_type{});
  step_barrier();  // the rings are reused below

  // ---- epilogue: the streams' partial results meet in LDS, rows go through a stage of LDS to
  // 16-byte nontemporal stores
  uint16_t* op = static_cast<uint16_t*>(a.out);
  const float l_tot = pair_sum(l_run);
  uint8_t* const stage_o = lds + (KS == 1 ? 0 : kKBytes) + wave_r * 32 * L::ROW;
  static_assert(KS > 1 || ROWS * L::ROW <= kKBytes + kVBytes, "the rings hold the rows");
  auto stage = [&](int dt, int i4, f32x4 x, float inv) {
    bf16x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(x[e] * inv);
    *reinterpret_cast<bf16x4*>(stage_o + L::k_pos(lane % 32, 4 * dt + i4) + 8 * half) = w;
  };
  float m_all = m_run, l_all = l_tot;
  if constexpr (KS == 1) {
    const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i4 = 0; i4 < 4; ++i4)
        stage(dt, i4, f32x4{o[dt][4 * i4], o[dt][4 * i4 + 1], o[dt][4 * i4 + 2], o[dt][4 * i4 + 3]}, inv);
  } else {
    // a unit is 8 of a lane's 32 values of O (dt, pair of i4); stream j owns units
    // [4 j / KS, 4 (j + 1) / KS), the others hand it theirs, scaled to the rows' common max
    constexpr int OWN = 4 / KS, SLOTS = KS == 2 ? 2 : 4;  // units per owner, slots per wave
    static_assert(kR32Waves * SLOTS * 2048 <= kKBytes && RW * 32 * L::ROW <= kVBytes, "the rings hold the exchange and the rows");
    float* const m_of = reinterpret_cast<float*>(table);  // [wave][32 rows]
    float* const l_of = m_of + kR32Waves * 32;
    if (half == 0) {
      m_of[wave * 32 + lane] = m_run;
      l_of[wave * 32 + lane] = l_tot;
    }
    __syncthreads();
    float m[KS];
#pragma unroll
    for (int j = 0; j < KS; ++j) {
      m[j] = m_of[(j * RW + wave_r) * 32 + lane % 32];
      m_all = fmaxf(m_all, m[j]);
    }
    l_all = 0.f;
    auto weight = [&](float mj) { return mj == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mj - m_all) * c); };
#pragma unroll
    for (int j = 0; j < KS; ++j) l_all = fmaf(weight(m[j]), l_of[(j * RW + wave_r) * 32 + lane % 32], l_all);
    const float w = weight(m_run);
    auto slot = [&](int of_wave, int u, int x) {  // 16 bytes a lane: half x of wave of_wave's unit u
      return reinterpret_cast<f32x4*>(lds) + ((of_wave * SLOTS + u % SLOTS) * 2 + x) * kWave + lane;
    };
    auto mine = [&](int u, int x) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[u / 2][8 * (u % 2) + 4 * x + e] * w;
      return v;
    };
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (wave_live && u / OWN != stream) {  // wave-uniform
#pragma unroll
        for (int x = 0; x < 2; ++x) *slot(wave, u, x) = mine(u, x);
      }
    __syncthreads();
    const float inv = l_all > 0.f ? 1.0f / l_all : 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (wave_live && u / OWN == stream) {
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          f32x4 v = mine(u, x);
#pragma unroll
          for (int j = 1; j < KS; ++j) v += *slot(((stream + j) % KS) * RW + wave_r, u, x);
          stage(u / 2, 2 * (u % 2) + x, v, inv);
        }
      }
  }
  __syncthreads();
  const int row = wrow + lane % 32;
  if (a.lse && stream == 0 && lane < 32 && row < row_end)
    a.lse[static_cast<int64_t>(h) * a.lq + row] = l_all > 0.f ? (m_all * c + __log2f(l_all)) * kLn2 : -INFINITY;
#pragma unroll
  for (int i = 0; i < 32 * L::CHUNKS / kWave / KS; ++i) {
    const int cid = stream * kWave + lane + i * KS * kWave;
    const int r = cid / L::CHUNKS, ch = cid % L::CHUNKS;
    if (wrow + r < row_end)
      __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(stage_o + L::k_pos(r, ch)),
                                  reinterpret_cast<u32x4*>(op + (static_cast<int64_t>(wrow + r) * a.H + h) * D + ch * 8));
  }
}

// ------------------------------------------------------------------ bf16 / MFMA, 64 rows per wave
// d = 128.  Four waves (one per SIMD) x 64 query rows, as two 32-row halves that share every
// K and V operand read from LDS: each 1 KB operand fragment feeds two MFMAs, half the
// LDS bytes per flop of 32 rows per wave, whose operand traffic equals the LDS
// bandwidth at the MFMA peak.  With one wave per SIMD the matrix core is kept busy
// from inside the wave: the instruction stream alternates MFMAs of one half with
// the softmax VALU work of the other (QK of half 1 with the exponentials of half
// 0, PV of half 0 with the exponentials of half 1), and MFMAs run asynchronously.
// The running max starts as the first tile's own max and may then lag the true one:
// O and l are rescaled only when exponentials against the stale max could exceed 2^8,
// well inside fp32 and bf16 range, and the final normalisation cancels the stale max
// exactly.
constexpr int kR64Waves = 4;
constexpr float kSlackSum = 256.0f;  // 2^8: how far exponentials may exceed 1 before O is rescaled
constexpr float kNoMax = -1.0e30f;   // running max before the first tile: finite, below any score

// Pins values at this point of the instruction stream: the exponentials of one half
// are computed between the other half's MFMAs, not moved down past the check that
// follows them to their first use.
__device__ __forceinline__ void keep_here(const bf16x8 (&pb)[4], float l) {
  asm volatile("" ::"v"(pb[0]), "v"(pb[1]), "v"(pb[2]), "v"(pb[3]), "v"(l));
}

// P V product with its accumulator in AccVGPRs.  Selected by the compiler, every
// MFMA accumulator sits in the VGPRs that the softmax VALU work also uses, and an
// MFMA writing its result there slows that work down; the asm keeps O in AccVGPRs.
// The asm also hides the MFMA from the compiler's hazard checks, so the wait states
// are explicit: two before the MFMA (any operand may have been written by VALU code
// just before it: a rematerialised constant, a copy out of a spill), the callers
// keep the A and B operands unchanged until the MFMA has read them (it reads them
// over its passes), and VALU code touches the accumulators only after
// acc_settled().
__device__ __forceinline__ void pv_mfma(f32x16& acc, const bf16x8& v, const bf16x8& p) {
  asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(v), "v"(p));
}
// The same MFMA with its two wait states filled by the softmax stream's own work, ahead of
// it: t = s c - m (the exponent of a score), and sum += u (an earlier exponential, taken
// more than the one wait state a transcendental's result needs before) or the other half's
// exponent.  The scores were formed an MFMA run earlier, so the VALU reads of MFMA results
// that the compiler does not see here are far past their hazard.  Against two empty wait
// states before every MFMA, 12 heads x 4,680 rows x 64 blocks: 113.2 -> 110.5 us; 5 heads x
// 3 groups x 1,560 rows in two key streams: 64.1 -> 61.7 us.
__device__ __forceinline__ void pv_mfma(f32x16& acc, const bf16x8& v, const bf16x8& p, float& t, float s, float c,
                                        float m, float& sum, float u) {
  asm volatile(
      "v_fma_f32 %1, %5, %6, -%7\n\tv_add_f32 %2, %2, %8\n\tv_mfma_f32_32x32x16_bf16 %0, %3, %4, %0"
      : "+a"(acc), "=&v"(t), "+v"(sum)
      : "v"(v), "v"(p), "v"(s), "v"(c), "v"(m), "v"(u));
}
__device__ __forceinline__ void pv_mfma(f32x16& acc, const bf16x8& v, const bf16x8& p, float& t, float s, float c,
                                        float m) {
  asm volatile("v_fma_f32 %1, %4, %5, -%6\n\ts_nop 0\n\tv_mfma_f32_32x32x16_bf16 %0, %2, %3, %0"
               : "+a"(acc), "=&v"(t)
               : "v"(v), "v"(p), "v"(s), "v"(c), "v"(m));
}
// Sixteen wait states (more than an 8-pass MFMA result needs) before VALU code reads
// or writes the accumulators; they pass through the asm so that no access moves
// ahead of it.
__device__ __forceinline__ void acc_settled(f32x16 (&o)[4]) {
  asm volatile("s_nop 7\n\ts_nop 7" : "+a"(o[0]), "+a"(o[1]), "+a"(o[2]), "+a"(o[3]));
}

// KS key streams: the workgroup's waves are KS sets of 4 / KS row waves, set j walking
// tiles j, j + KS, ... of the list and the sets meeting in LDS at the end, for grids that
// would leave CUs idle with 256 rows per workgroup.
template <int KS>
__global__ __launch_bounds__(kR64Waves* kWave, 1) void k_attn_bf16_r64(AttnArgs a) {
  constexpr int D = 128;
  using L = KeyTileLds<D>;
  constexpr int NT = kR64Waves * kWave;
  constexpr int RW = kR64Waves / KS;  // row waves per stream
  constexpr int ROWS = RW * 64;
  constexpr int DT = D / 32;
  constexpr int KK = D / 16;
  constexpr int DMA_PER_WAVE = L::TILE / 1024 / RW;  // 1 KB DMA instructions per wave and tile, K and V each
  // Four stages of K and V for one stream (128 KB), tile t in stage t mod 4:
  // iteration t reads the K of tile t and the V of tile t - 1 while tile t + 1 has landed
  // and tile t + 2 arrives in the stage of tile t - 2.
  // Two a stream for two streams: iteration t reads the K of tile t and the V of tile t - 1
  // while the K of tile t + 1 and the V of tile t arrive in the stages that iteration t - 1
  // has read.
  constexpr bool kDeep = KS == 1;
  constexpr int kStages = kDeep ? 4 : 2;
  constexpr int kRing = KS * kStages * L::TILE;
  __shared__ __attribute__((aligned(1024))) uint8_t k_ring[kRing];
  __shared__ __attribute__((aligned(1024))) uint8_t v_ring[kRing];
  __shared__ __attribute__((aligned(16))) int2 table[2 * NT];
  __shared__ int scan_tmp[kR64Waves];

  int h, hr, row0, row_end;
  resolve_tile(a, xcd_contiguous_id(blockIdx.x, gridDim.x), ROWS, h, hr, row0, row_end);
  if (row0 >= row_end) return;  // workgroup-uniform: no barrier has been reached
  const int32_t* list;
  int count;
  resolve_list(a, hr, list, count);

  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int wave_r = KS == 1 ? wave : wave % RW, stream = KS == 1 ? 0 : wave / RW;
  // this thread's entry of the first decoded stretch, read without waiting for the
  // count (the list holds top_k entries)
  const int id0 = list != nullptr && tid < a.top_k ? list[tid] : INT_MIN;
  const int half = lane / 32;
  const uint16_t* qp = static_cast<const uint16_t*>(a.q);
  const uint16_t* kp = static_cast<const uint16_t*>(a.k_pages);
  const uint16_t* vp = static_cast<const uint16_t*>(a.v_pages);

  // Q^T B operands of the two halves: lane holds query wrow + 32 g + lane % 32
  const float c = a.scale * kLog2e;  // scores to the softmax's log2 units, applied in fp32
  const int wrow = row0 + wave_r * 64;
  const bool wave_live = wrow < row_end;  // wave-uniform
  // the Q rows are loaded here and moved to AccVGPRs once the first tiles' DMA is
  // issued, so that their latency overlaps the block-list decode
  uint4 qx0[KK], qx1[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    const int r0 = wrow + lane % 32, r1 = r0 + 32;
    qx0[kk] = qx1[kk] = make_uint4(0, 0, 0, 0);
    if (r0 < row_end)
      qx0[kk] = *reinterpret_cast<const uint4*>(qp + (static_cast<int64_t>(r0) * a.H + h) * D + 16 * kk + 8 * half);
    if (r1 < row_end)
      qx1[kk] = *reinterpret_cast<const uint4*>(qp + (static_cast<int64_t>(r1) * a.H + h) * D + 16 * kk + 8 * half);
  }
  bf16x8 q0[KK], q1[KK];

  f32x16 o0[DT], o1[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      o0[dt][i] = 0.f;
      o1[dt][i] = 0.f;
    }
  // running max in scaled log2 units (max * scale * log2 e) and this lane's share of l
  float ms0 = kNoMax, ms1 = kNoMax, l0 = 0.f, l1 = 0.f;

  // ---- tile sequence: (page, sub-tile << 8 | valid keys), from the decoded table
  int next_entry = 0, ntab = 0, ti = 0;
  // The next table entry as read from LDS (the same in every lane; made scalar where
  // used, so that the read's latency is not waited for here).  Called by every thread
  // together: it refills the table (with barriers) when it runs out.
  // With several streams every stream takes its own of the next KS entries (an empty tile
  // past the table's end), and `more` tells whether there was one for any of them.
  bool more = false;
  auto next_tile_raw = [&]() -> int2 {
    if (KS == 1 ? ti == ntab : ti >= ntab) {
      ntab = 0;
      ti = 0;
      while (ntab == 0 && next_entry < count) {
        ntab = decode_tiles<NT>(a, head_table(a, h), list, count, next_entry, table, scan_tmp,
                                next_entry == 0 ? id0 : INT_MIN);
        next_entry += NT;
      }
      if (KS > 1) ntab = __builtin_amdgcn_readfirstlane(ntab);
      if (ntab == 0) {  // past the end: an empty tile
        more = false;
        return make_int2(0, 0);
      }
    }
    if constexpr (KS == 1) return table[ti++];
    more = true;
    const int2 m = ti + stream < ntab ? table[ti + stream] : make_int2(0, 0);
    ti += KS;
    return m;
  };
  auto scalar_tile = [](int2 m) {
    return make_int2(__builtin_amdgcn_readfirstlane(m.x), __builtin_amdgcn_readfirstlane(m.y));
  };
  // this lane's source offsets for its DMA instructions (instruction m = wave_r + RW i of the tile)
  int k_src[DMA_PER_WAVE], v_src[DMA_PER_WAVE];
#pragma unroll
  for (int i = 0; i < DMA_PER_WAVE; ++i) {
    const int r = L::DMA_ROWS * (wave_r + RW * i) + lane / L::CHUNKS, p = lane % L::CHUNKS;
    k_src[i] = L::k_pos(r, p);
    v_src[i] = L::v_pos(r, p);
  }
  const int wave_s = __builtin_amdgcn_readfirstlane(wave_r);  // scalar copies: LDS destinations go to M0
  const int ring0 = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(stream) * kStages * L::TILE;  // this stream's stages
  // Scalar bases: this head's slab of page 0, the page stride, and the wave's first
  // LDS destination.  Everything about a tile's DMA is then a few scalar ops.
  const int64_t h_elems = static_cast<int64_t>(__builtin_amdgcn_readfirstlane(h)) * a.B * D;
  const uint16_t* const kp_h = kp + h_elems;
  const uint16_t* const vp_h = vp + h_elems;
  const int64_t page_elems = static_cast<int64_t>(a.H) * a.B * D;
  const uint32_t m0_k = lds_offset(k_ring) + ring0 + wave_s * 1024, m0_v = lds_offset(v_ring) + ring0 + wave_s * 1024;
  auto slab_of = [&](int2 m) { return static_cast<int64_t>(m.x) * page_elems + static_cast<int64_t>(m.y >> 8) * kTileKeys * D; };
  // instruction i of the DMA of tile mk's K into stage sk and of tile mv's V into stage sv
  // (empty tiles load nothing and write zeros); the tiles are the same in every lane.  The
  // LDS bases pass through an empty asm so that each destination is formed where it is
  // used: hoisted out of the loop, the 32 stage/instruction combinations would each hold
  // a scalar register.
  auto issue_part = [&](int2 mk, int sk, int2 mv, int sv, int i) {
    const u32x4 kr = buffer_rsrc(kp_h + slab_of(mk), (mk.y & 255) * D * 2),
                vr = buffer_rsrc(vp_h + slab_of(mv), (mv.y & 255) * D * 2);
    uint32_t dk = m0_k, dv = m0_v;
    asm volatile("" : "+s"(dk), "+s"(dv));
    dma_16x64(kr, k_src[i], dk + sk * L::TILE + RW * i * 1024);
    dma_16x64(vr, v_src[i], dv + sv * L::TILE + RW * i * 1024);
  };
  auto issue = [&](int2 mk, int sk, int2 mv, int sv) {
#pragma unroll
    for (int i = 0; i < DMA_PER_WAVE; ++i) issue_part(mk, sk, mv, sv, i);
  };

  // keys past the block's end of a partial tile get -inf scores (the key base goes
  // through an empty asm so that none of this is computed ahead of the rare branch)
  auto mask_tail = [&](f32x16 (&s)[2], int nvalid) {
    int kb = 8 * half;
    asm volatile("" : "+v"(kb));
#pragma unroll
    for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = 32 * t2 + (i < 8 ? kb + i : 16 + kb + (i - 8));
        if (key >= nvalid) s[t2][i] = -INFINITY;
      }
  };
  // A half's softmax as a stream over its 32 S elements per lane (element E is
  // s[E / 16][E % 16]; it lands in P^T fragment E / 8 at position E % 8).  Slot g
  // forms the exponent c s - max of element g (one fma: the scale is applied in
  // fp32), takes the exponential of element g - 1, adds element g - 2 to the row sum
  // and, on odd slots, packs elements g - 3 and g - 2 into P (late enough for the PV
  // run that carries the early slots to have read the previous tile's P fragment 0).
  // No op of a slot reads a result of the same slot, so a slot placed next to one
  // MFMA issues without waiting on VALU latency; slots 32 and 33 finish the stream.
  // Each result goes through an empty asm so that the IR passes keep it in its slot
  // (they would otherwise sink every op next to its first use).  The row sum is taken
  // over the fp32 values.
  // `formed`, `added`: the exponent, the sum have been taken by the slot's PV MFMA.
  auto soft_slot = [&](const f32x16 (&s)[2], float ms, float& acc, bf16x8 (&pb)[4], float (&tq)[32],
                       float (&uq)[32], int g, bool formed = false, bool added = false) {
    if (g < 32 && !formed) {
      tq[g] = fmaf(s[g / 16][g % 16], c, -ms);
      asm volatile("" : "+v"(tq[g]));
    }
    if (g >= 1 && g <= 32) {
      uq[g - 1] = __builtin_amdgcn_exp2f(tq[g - 1]);
      asm volatile("" : "+v"(uq[g - 1]));
    }
    if (g >= 2 && g <= 33 && !added) {
      acc += uq[g - 2];
      asm volatile("" : "+v"(acc));
    }
    if (g % 2 == 1 && g >= 3 && g <= 33) {
      const int e = g - 3;
      bf16x2 pk = {static_cast<__bf16>(uq[e]), static_cast<__bf16>(uq[e + 1])};
      asm volatile("" : "+v"(pk));
      pb[e / 8][e % 8] = pk[0];
      pb[e / 8][e % 8 + 1] = pk[1];
    }
  };
  const int krow = s_row_perm(lane % 32);
  typedef __attribute__((address_space(3))) i16x4 lds_i16x4;
  // Operand fragments, read from LDS ahead of the MFMAs that use them: K fragments four
  // ahead, V fragments three (four would take the PV run past 256 VGPRs).
  // The lane's part of each address is fixed for the whole loop (8 K and 4 V byte
  // offsets, the chunk permutations depending only on the lane); the stage, the key
  // group and the ring base are compile-time constants that fold into the reads'
  // offset fields.
  // (masked to the 18 bits of the LDS address space, which lets the compiler see that
  // base + constant cannot wrap)
  uint32_t k_lane[KK], v_lane[DT];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_lane[kk] = (lds_offset(k_ring) + ring0 + L::k_pos(krow, 2 * kk + half)) & 0x3ffffu;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    const int key0 = 8 * half + (lane % 16) / 4;
    const int ch = 4 * dt + 2 * ((lane / 16) % 2) + (lane % 4) / 2;
    v_lane[dt] = (lds_offset(v_ring) + ring0 + L::v_pos(key0, ch) + 8 * (lane % 2)) & 0x3ffffu;
  }
  typedef __attribute__((address_space(3))) const uint8_t lds_u8;
  auto k_frag = [&](int st, int f) {  // f = 8 t2 + kk: keys 32 t2 .., k-step kk
    lds_u8* p = reinterpret_cast<lds_u8*>(static_cast<uintptr_t>(k_lane[f % KK])) + (st * L::TILE + (f / KK) * 32 * L::ROW);
    return *reinterpret_cast<__attribute__((address_space(3))) const bf16x8*>(p);
  };
  auto v_frag = [&](int st, int f) {  // f = 4 j + dt: keys 16 j .., d 32 dt ..; two transposing reads (keys +4)
    lds_u8* p = reinterpret_cast<lds_u8*>(static_cast<uintptr_t>(v_lane[f % DT])) + (st * L::TILE + (f / DT) * 16 * L::ROW);
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p + 4 * L::ROW));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  // The exponentials of a half are computed against its running max before the
  // tile's own max is known (the first tile's against its own max, taken once).  They
  // stand (every p <= 2^8) unless some lane's sum of them exceeds 2^8 or overflowed,
  // which takes a rise of the max by more than 3 log2 units; only then is the tile's S
  // formed again from the K still in LDS (stage kst, nvalid keys), its max taken, O
  // and l moved to the new max and the exponentials redone.  The next tile's
  // exponentials are formed after this point, against the new max.  The rare path is
  // laid out away from the loop, which then runs straight through.  With two stages the
  // tile's K is already being replaced: it is read from memory again, in the operand
  // layout (tile m; rows past its valid keys read as zero).
  auto settle = [&](float& ms, float& l, float acc, f32x16 (&o)[DT], bf16x8 (&pb)[4], const bf16x8 (&q)[KK], int kst,
                    int2 m) {
    if (__builtin_expect(__any(acc > kSlackSum), 0)) {
      const int nvalid = m.y & 255;
      const u32x4 r = buffer_rsrc(kp_h + slab_of(m), nvalid * D * 2);
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
          reinterpret_cast<void*>(static_cast<uint64_t>(r[1]) << 32 | r[0]), 0, r[2], r[3]);
      int at = krow * L::ROW + 16 * half;
      asm volatile("" : "+v"(at));
      f32x16 s[2];
#pragma unroll
      for (int f = 0; f < 2 * KK; ++f) {
        bf16x8 k;
        if constexpr (kDeep)
          k = k_frag(kst, f);
        else
          k = __builtin_bit_cast(
              bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at + 32 * (f % KK), (f / KK) * 32 * L::ROW, 0));
        s[f / KK] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k, q[f % KK], f % KK ? s[f / KK] : f32x16{}, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // one fragment at a time: this path must not raise register use
      }
      if (nvalid < kTileKeys) mask_tail(s, nvalid);
      float m0 = fmaxf(s[0][0], s[1][0]), m1 = fmaxf(s[0][1], s[1][1]);
#pragma unroll
      for (int i = 2; i < 16; i += 2) {
        m0 = fmaxf(m0, fmaxf(s[0][i], s[1][i]));
        m1 = fmaxf(m1, fmaxf(s[0][i + 1], s[1][i + 1]));
      }
      const float m_new = fmaxf(ms, pair_max(fmaxf(m0, m1)) * c);
      const float alpha = __builtin_amdgcn_exp2f(ms - m_new);
      l *= alpha;
      acc_settled(o);
      // one 16-register block at a time through VGPRs (O stays in AccVGPRs)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        f32x16 t = o[dt];
        asm volatile("" : "+v"(t));
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] *= alpha;
        o[dt] = t;
        asm volatile("" : "+a"(o[dt]));
      }
      ms = m_new;
      acc = 0.f;
#pragma unroll
      for (int e = 0; e < 32; e += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(s[e / 16][e % 16], c, -m_new));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(s[e / 16][e % 16 + 1], c, -m_new));
        acc += p0 + p1;
        pb[e / 8][e % 8] = static_cast<__bf16>(p0);
        pb[e / 8][e % 8 + 1] = static_cast<__bf16>(p1);
      }
    }
    l += acc;
  };

  // ---- Software pipeline over tiles.  Iteration t runs two runs of 32 MFMAs, each
  // MFMA carrying one softmax stream slot (one exponential, a half-rate VALU op, and
  // two or three other VALU ops fill the MFMA shadow only when spread this thin):
  //   QK run  S of tile t, both halves (each K fragment feeds the two halves' MFMAs
  //           back to back); slots 15-33 of tile t-1's two streams; DMA of tile t+2
  //   PV run  O += P V of tile t-1, both halves (each V^T fragment feeds two MFMAs);
  //           slots 0-14 of tile t's two streams
  // with both halves' softmax checks of tile t-1 between the runs.  Operand fragments
  // are read just in time, so the registers hold S of two tiles and P of one.  One
  // barrier per iteration, at its end: tile t+1 has landed and every wave is past its
  // reads of the stages that the next iteration's DMA refills.  "Tile -1" is an
  // all-masked dummy (S = -inf, P = 0, its V stage DMA'd from an empty tile: zeros),
  // and the sequence ends with one empty tile whose iteration finishes the last one.
  constexpr int NRUN = 4 * KK;          // MFMAs per run (both halves)
  constexpr int FIRST = NRUN / 2 - 1;   // slots that ride on the PV run
  constexpr int TAIL = FIRST + NRUN / 2;
  static_assert(4 * DT == NRUN / 2 && 2 * KK == NRUN / 2, "QK and PV runs of one length");
  constexpr int DMA_EVERY = NRUN / DMA_PER_WAVE, DMA_AT = DMA_EVERY == 8 ? 5 : DMA_EVERY / 2;
  f32x16 sa0[2], sa1[2], sb0[2], sb1[2];
  bf16x8 pb0[4], pb1[4];
  // the first tile's max of a half's S in scaled log2 units, from both lanes of each
  // row (masked keys are -inf: with no valid key at all it stays kNoMax)
  bool first_tile = true;
  auto tile_max = [&](const f32x16 (&s)[2]) {
    float m0 = fmaxf(s[0][0], s[1][0]), m1 = fmaxf(s[0][1], s[1][1]);
#pragma unroll
    for (int i = 2; i < 16; i += 2) {
      m0 = fmaxf(m0, fmaxf(s[0][i], s[1][i]));
      m1 = fmaxf(m1, fmaxf(s[0][i + 1], s[1][i + 1]));
    }
    return fmaxf(kNoMax, pair_max(fmaxf(m0, m1)) * c);
  };
  float acc0 = 0.f, acc1 = 0.f;
  // the two halves' softmax streams (only a few elements of each are live at a time)
  float tq0[32], uq0[32], tq1[32], uq1[32];
#pragma unroll
  for (int t2i = 0; t2i < 2; ++t2i)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      sa0[t2i][i] = -INFINITY;
      sa1[t2i][i] = -INFINITY;
    }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    pb0[j] = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
    pb1[j] = pb0[j];
  }
  tq0[FIRST - 1] = tq1[FIRST - 1] = -INFINITY;  // the dummy tile's streams enter the loop at slot FIRST
  uq0[FIRST - 3] = uq0[FIRST - 2] = uq1[FIRST - 3] = uq1[FIRST - 2] = 0.f;
  const int2 empty = make_int2(0, 0);
  int2 prev = empty;

  int2 cur = scalar_tile(next_tile_raw());
  bool cur_more = more, t1_more = false;  // whether any stream has a tile t, t + 1
  int2 t1 = empty;
  if constexpr (kDeep) {
    t1 = scalar_tile(next_tile_raw());
    t1_more = more;
    issue(empty, kStages - 1, empty, kStages - 1);  // V of tile -1
    issue(cur, 0, cur, 0);
    issue(t1, 1, t1, 1);
  } else {
    issue(cur, 0, empty, 1);  // K of tile 0, V of tile -1
  }
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    q0[kk] = __builtin_bit_cast(bf16x8, qx0[kk]);
    q1[kk] = __builtin_bit_cast(bf16x8, qx1[kk]);
    // Q lives in AccVGPRs next to O; the VGPRs hold S, P and the operand fragments
    asm volatile("" : "+a"(q0[kk]), "+a"(q1[kk]));
  }
  // The Q loads and the block-list reads have landed (the compiler waited for them
  // before the decode and the scaling, so it knows of no load of its own pending in
  // the loop, where any wait it inserted would also drain the DMA in flight, which it
  // does not see); of the DMA, the dummy stage and tile 0 must land before the loop,
  // tile 1 may still be in flight.
  constexpr int IN_FLIGHT = kDeep ? 2 * DMA_PER_WAVE : 0;
  __builtin_amdgcn_s_waitcnt(vmcnt_only(IN_FLIGHT));
  lds_barrier();

  // The operands of the PV MFMA issued last, held until it has read them: those of a run's
  // last one until the next iteration's QK run has begun (waiting for it at the run's end
  // took 1% of a tile).
  bf16x8 hold_a = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0)), hold_b = hold_a;

  // Iteration t (t mod kStages = T, a compile-time constant, as are the stages) with tile
  // t-1's S in (so0, so1) and tile t's formed in (sn0, sn1); consecutive iterations
  // swap the two, so that no S is ever copied.  Returns false after the iteration of
  // the empty tile that ends the sequence.
  auto iteration = [&](f32x16 (&so0)[2], f32x16 (&so1)[2], f32x16 (&sn0)[2], f32x16 (&sn1)[2], auto tmod) {
    constexpr int T = decltype(tmod)::value;
    constexpr int kst = T, vst = (T + kStages - 1) % kStages;
    constexpr int k_into = kDeep ? (T + 2) % kStages : vst, v_into = kDeep ? k_into : T;
    bf16x8 kf[2 * KK], vf[4 * DT];
    if (wave_live) {
      kf[0] = k_frag(kst, 0);
      kf[1] = k_frag(kst, 1);
      kf[2] = k_frag(kst, 2);
      kf[3] = k_frag(kst, 3);
    }
    const int2 t2 = scalar_tile(next_tile_raw());  // every thread; refills the table at its end
    const int2 v_tile = kDeep ? t2 : cur;          // the tiles whose K and V arrive during this iteration: t2 and this
    const int cur_nvalid = cur.y & 255;
    if (wave_live) {
      // ---- QK run
#pragma unroll
      for (int i = 0; i < NRUN; ++i) {
        const int f = i / 2;
        if (i % 2 == 0) {
          sn0[f / KK] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[f], q0[f % KK], f % KK ? sn0[f / KK] : f32x16{}, 0, 0, 0);
        } else {
          sn1[f / KK] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[f], q1[f % KK], f % KK ? sn1[f / KK] : f32x16{}, 0, 0, 0);
        }
        if (i % 2 == 0) soft_slot(so0, ms0, acc0, pb0, tq0, uq0, FIRST + f);
        if (i % 2 == 1) soft_slot(so1, ms1, acc1, pb1, tq1, uq1, FIRST + f);
        if (i % 2 == 0 && f + 4 < 2 * KK) kf[f + 4] = k_frag(kst, f + 4);
        if (i == 1) asm volatile("" ::"v"(hold_a), "v"(hold_b));  // the previous PV run's last operands
        if (i % DMA_EVERY == DMA_AT) issue_part(t2, k_into, v_tile, v_into, i / DMA_EVERY);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int g = TAIL; g < 34; ++g) {
        soft_slot(so0, ms0, acc0, pb0, tq0, uq0, g);
        soft_slot(so1, ms1, acc1, pb1, tq1, uq1, g);
      }
      keep_here(pb0, acc0);
      keep_here(pb1, acc1);
      vf[0] = v_frag(vst, 0);
      vf[1] = v_frag(vst, 1);
      vf[2] = v_frag(vst, 2);
      settle(ms0, l0, acc0, o0, pb0, q0, vst, prev);
      settle(ms1, l1, acc1, o1, pb1, q1, vst, prev);
      acc0 = 0.f;
      acc1 = 0.f;
      if (__builtin_expect(cur_nvalid < kTileKeys, 0)) {
        mask_tail(sn0, cur_nvalid);
        mask_tail(sn1, cur_nvalid);
      }
      if (T == 0 && first_tile) {  // the first tile's exponentials use its own max
        first_tile = false;
        ms0 = tile_max(sn0);
        ms1 = tile_max(sn1);
      }
      // ---- PV run.  Stream slot (g, half) of tile t rides on MFMA 2 g + half + 2, past the
      // last MFMA that reads the previous tile's P fragment it overwrites.
      // An MFMA reads its A and B registers over its passes, so each MFMA's operands
      // are held (an empty asm use) until the end of the next slot, when it has
      // finished: the compiler, which does not see these MFMAs, would otherwise give
      // the registers to the next value as soon as the MFMA is issued.
#pragma unroll
      for (int i = 0; i < NRUN; ++i) {
        const int f = i / 2;
        const bf16x8 op_a = vf[f], op_b = i % 2 ? pb1[f / DT] : pb0[f / DT];
        f32x16& o = i % 2 ? o1[f % DT] : o0[f % DT];
        const int g = f - 1;  // the slot that rides on this MFMA
        if (i < 2)
          pv_mfma(o, op_a, op_b);
        else if (g < 2)
          pv_mfma(o, op_a, op_b, i % 2 ? tq1[g] : tq0[g], (i % 2 ? sn1 : sn0)[g / 16][g % 16], c, i % 2 ? ms1 : ms0);
        else
          pv_mfma(o, op_a, op_b, i % 2 ? tq1[g] : tq0[g], (i % 2 ? sn1 : sn0)[g / 16][g % 16], c, i % 2 ? ms1 : ms0,
                  i % 2 ? acc1 : acc0, i % 2 ? uq1[g - 2] : uq0[g - 2]);
        if (i % 2 == 0 && f + 3 < 4 * DT) vf[f + 3] = v_frag(vst, f + 3);
        if (i >= 2) {
          if (i % 2 == 0) soft_slot(sn0, ms0, acc0, pb0, tq0, uq0, g, true, true);
          if (i % 2 == 1) soft_slot(sn1, ms1, acc1, pb1, tq1, uq1, g, true, true);
        }
        if (i > 0) asm volatile("" ::"v"(hold_a), "v"(hold_b));
        hold_a = op_a;
        hold_b = op_b;
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      issue(t2, k_into, v_tile, v_into);
    }
    // ---- what iteration t+1 reads has landed (with four stages the DMA of tile t+2 may
    // still be in flight) and every wave is past its reads of the stages refilled next
    __builtin_amdgcn_s_waitcnt(vmcnt_only(IN_FLIGHT));
    lds_barrier();
    prev = cur;
    const bool go_on = KS == 1 ? cur_nvalid != 0 : cur_more;
    cur = kDeep ? t1 : t2;
    cur_more = kDeep ? t1_more : more;
    t1 = t2;
    t1_more = more;
    return go_on;
  };
  for (;;) {
    if (!iteration(sa0, sa1, sb0, sb1, std::integral_constant<int, 0>{})) break;
    if (!iteration(sb0, sb1, sa0, sa1, std::integral_constant<int, 1>{})) break;
    if constexpr (kStages == 4) {
      if (!iteration(sa0, sa1, sb0, sb1, std::integral_constant<int, 2>{})) break;
      if (!iteration(sb0, sb1, sa0, sa1, std::integral_constant<int, 3>{})) break;
    }
  }
  asm volatile("s_nop 7\n\ts_nop 3" ::"v"(hold_a), "v"(hold_b));
  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));  // no DMA may land in the stages reused below
  __syncthreads();

  // ---- epilogue: normalise, stage O through LDS (one 16 KB stage per wave, chunks
  // permuted like K), store rows with 16-byte nontemporal writes (each row is written
  // once, and the L2 then holds no dirty lines of O for the end of the kernel to
  // write back)
  constexpr int STAGE = 64 * L::ROW;  // 64 rows per wave
  uint16_t* op = static_cast<uint16_t*>(a.out);
  auto store_rows = [&](const uint8_t* stage_o) {  // the wave's share of its rows' chunks
#pragma unroll
    for (int i = 0; i < 64 * L::CHUNKS / kWave / KS; ++i) {
      const int cid = stream * kWave + lane + i * KS * kWave;
      const int r = cid / L::CHUNKS, ch = cid % L::CHUNKS;
      const int qrow = wrow + r;
      if (qrow < row_end)
        __builtin_nontemporal_store(*reinterpret_cast<const u32x4*>(stage_o + L::k_pos(r, ch)),
                                    reinterpret_cast<u32x4*>(op + (static_cast<int64_t>(qrow) * a.H + h) * D + ch * 8));
    }
  };
  if constexpr (KS == 1) {
    uint8_t* const stage_o = k_ring + wave * STAGE;
    auto finish = [&](f32x16 (&o)[DT], float ms, float l, int g) {
      const float l_tot = pair_sum(l);
      const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.f;
      const int r = 32 * g + lane % 32;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          bf16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(o[dt][4 * i4 + e] * inv);
          // d = 32 dt + 8 i4 + 4 half: chunk 4 dt + i4, byte 8 half within it
          *reinterpret_cast<bf16x4*>(stage_o + L::k_pos(r, 4 * dt + i4) + 8 * half) = w;
        }
      const int qr = wrow + r;
      if (a.lse && lane < 32 && qr < row_end)
        a.lse[static_cast<int64_t>(h) * a.lq + qr] = l_tot > 0.f ? (ms + __log2f(l_tot)) * kLn2 : -INFINITY;
    };
    if (wave_live) {
      acc_settled(o0);
      acc_settled(o1);
      finish(o0, ms0, l0, 0);
      finish(o1, ms1, l1, 1);
    }
    __syncthreads();
    if (wave_live) store_rows(stage_o);
  } else {
    // The streams' partial results of a row wave's 64 rows meet in LDS.  A unit is 32 rows
    // (half g) x 32 of d (dt), 16 values a lane; every unit has an owner among the
    // streams, the others hand it theirs, scaled to the rows' common max.
    constexpr int UNITS = DT;  // slots for units handed over, per wave (4 KB each)
    static_assert(KS == 2, "a half of the rows per stream");
    static_assert(kR64Waves * UNITS * 4096 <= kRing && RW * STAGE <= kRing, "the rings hold the exchange and the output");
    float* const m_of = reinterpret_cast<float*>(table);  // [wave][64 rows]
    float* const l_of = m_of + kR64Waves * 64;
    static_assert(2 * kR64Waves * 64 * sizeof(float) <= sizeof(table), "the table holds the rows' max and sum");
    const float lt0 = pair_sum(l0), lt1 = pair_sum(l1);
    m_of[wave * 64 + lane] = half ? ms1 : ms0;
    l_of[wave * 64 + lane] = half ? lt1 : lt0;
    __syncthreads();
    float mt[2], lt[2], wt[2];  // per half: the row's max and sum over the streams, this stream's weight
#pragma unroll
    for (int g = 0; g < 2; ++g) {
      float m[KS];
      mt[g] = kNoMax;
#pragma unroll
      for (int j = 0; j < KS; ++j) {
        m[j] = m_of[(j * RW + wave_r) * 64 + 32 * g + lane % 32];
        mt[g] = fmaxf(mt[g], m[j]);
      }
      lt[g] = 0.f;
#pragma unroll
      for (int j = 0; j < KS; ++j)
        lt[g] = fmaf(__builtin_amdgcn_exp2f(m[j] - mt[g]), l_of[(j * RW + wave_r) * 64 + 32 * g + lane % 32], lt[g]);
      wt[g] = __builtin_amdgcn_exp2f((g ? ms1 : ms0) - mt[g]);
    }
    auto unit = [&](int w, int dt) {  // where wave w puts the unit of the other's half
      return reinterpret_cast<f32x4*>(k_ring) + ((w * UNITS + dt) * 4) * kWave + lane;
    };
    if (wave_live) {
      acc_settled(o0);
      acc_settled(o1);
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          if (stream != g) {  // wave-uniform
            f32x4* const to = unit(wave, dt);
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
              f32x4 x;
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = (g ? o1 : o0)[dt][4 * i4 + e] * wt[g];
              to[i4 * kWave] = x;
            }
          }
    }
    __syncthreads();
    uint8_t* const stage_o = v_ring + wave_r * STAGE;
    if (wave_live) {
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        const float inv = lt[g] > 0.f ? 1.0f / lt[g] : 0.f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          if (stream == g) {
#pragma unroll
            for (int i4 = 0; i4 < 4; ++i4) {
              f32x4 x;
#pragma unroll
              for (int e = 0; e < 4; ++e) x[e] = (g ? o1 : o0)[dt][4 * i4 + e] * wt[g];
#pragma unroll
              for (int j = 1; j < KS; ++j) {  // the other streams' in one order, from the next on
                const f32x4 y = unit(((stream + j) % KS) * RW + wave_r, dt)[i4 * kWave];
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] += y[e];
              }
              bf16x4 w;
#pragma unroll
              for (int e = 0; e < 4; ++e) w[e] = static_cast<__bf16>(x[e] * inv);
              *reinterpret_cast<bf16x4*>(stage_o + L::k_pos(32 * g + lane % 32, 4 * dt + i4) + 8 * half) = w;
            }
            const int qr = wrow + 32 * g + lane % 32;
            if (dt == 0 && a.lse && lane < 32 && qr < row_end)
              a.lse[static_cast<int64_t>(h) * a.lq + qr] = lt[g] > 0.f ? (mt[g] + __log2f(lt[g])) * kLn2 : -INFINITY;
          }
      }
    }
    __syncthreads();
    if (wave_live) store_rows(stage_o);
  }
}

// ------------------------------------------------------------------ fp32 / MFMA
// fp32 attention on v_mfma_f32_32x32x2_f32 (fp32 products and accumulation, 64 flops per
// cycle and SIMD): S^T = K Q^T, O^T += V^T P^T, as in the bf16 kernels.  The MFMAs bound
// it: a score costs 4 d flops, so the softmax is a twelfth of a tile's cycles at d = 128.
//  - A workgroup is 32 query rows of one (head, group); its waves split the keys, wave w
//    taking the 32-key tiles w, w + waves, ..., and meet in LDS at the end.  So the row
//    tile stays small (a 1,560-row frame of 12 heads gives 588 workgroups, a 256-row one of
//    2 heads 16 with their keys spread over every wave), no wave waits for another inside
//    the loop, and two workgroups share a CU.
//  - MFMA step (u, e) of the scores multiplies dimension 8 u + 4 half + e of both operands
//    (any bijection will do, as long as K and Q agree), so a lane's K and Q come 16 bytes
//    at a time.  K passes through the wave's own LDS tile: read from memory in the operand
//    layout, 64 separate 16-byte pieces a load, the vector cache was busy 62% of the time
//    and the frame below took 132 us instead of 117.
//  - Accumulator element i of lane l is key 8 (i / 4) + 4 half + i % 4, query l % 32: PV step
//    i takes P as it stands as the B operand and V rows 8 (i / 4) + 4 half + i % 4 as the
//    A operand, lane l % 32 = c supplying d = DT c + dt to accumulator dt with one load.
//  - K of the next tile is on its way while the PV MFMAs of this one run, V while the next
//    tile's QK MFMAs run: one copy of each.
// Against one lane per query row with its dot products and exponentials in series, at
// 12 heads x 1,560 rows x 1,024 keys, d = 128: 2,485 -> 114 us (84 TFLOP/s; 62 us at the
// rate of a large fp32 product, 82 us for the CUs that get three of the 588 workgroups; the
// MFMA pipe is busy for 73% of a busy CU's cycles);
// at 2 heads x 256 rows x 256 keys, d = 64: 292 -> 11 us.
constexpr int kF32Rows = 32;
constexpr int kF32Keys = 32;

// Waves per workgroup; 256 registers a wave allow two per SIMD.
template <int D>
struct F32Shape {
  static constexpr int NW = D == 128 ? 4 : 8;
  static constexpr int STRIDE = D + 4;  // LDS row of O, in floats: 16 rows cover the banks once
};

template <int D>
__global__ __launch_bounds__(F32Shape<D>::NW* kWave, 2) void k_attn_f32(AttnArgs a) {
  constexpr int NW = F32Shape<D>::NW, STRIDE = F32Shape<D>::STRIDE;
  constexpr int NT = NW * kWave;
  constexpr int U = D / 8;    // 16-byte K pieces per lane and tile
  constexpr int DT = D / 32;  // accumulators along d, floats per V load
  typedef float vdt __attribute__((ext_vector_type(DT)));
  __shared__ __attribute__((aligned(16))) float o_lds[NW * kF32Rows * STRIDE];
  __shared__ float m_lds[NW][kF32Rows], l_lds[NW][kF32Rows];
  __shared__ int2 table[2 * NT];
  __shared__ int scan_tmp[NW];

  int h, hr, row0, row_end;
  resolve_tile(a, a.first_wg + xcd_contiguous_id(blockIdx.x, gridDim.x), kF32Rows, h, hr, row0, row_end);
  if (row0 >= row_end) return;  // workgroup-uniform: no barrier has been reached
  const int32_t* list;
  int count;
  resolve_list(a, hr, list, count);
  const int tid = threadIdx.x, lane = tid % kWave, half = lane / 32, col = lane % 32;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const float* qp = static_cast<const float*>(a.q);
  const float* kp = static_cast<const float*>(a.k_pages);
  const float* vp = static_cast<const float*>(a.v_pages);

  f32x4 q[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    q[u] = f32x4{};
    if (row0 + col < row_end)
      q[u] = *reinterpret_cast<const f32x4*>(qp + (static_cast<int64_t>(row0 + col) * a.H + h) * D + 8 * u + 4 * half);
  }
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;  // max of scale * <q, k>, this lane's share of l

  vdt vr[16];
  // Tile t of the table's 64-key entries halved: the element offset of its first key and
  // its valid keys.
  auto tile_of = [&](int t, int64_t& off) -> int {
    const int2 e = table[t / 2];
    const int page = __builtin_amdgcn_readfirstlane(e.x), meta = __builtin_amdgcn_readfirstlane(e.y);
    const int s = t % 2;
    off = ((static_cast<int64_t>(page) * a.H + h) * a.B + (meta >> 8) * kTileKeys + s * kF32Keys) * D;
    const int nv = (meta & 255) - s * kF32Keys;
    return nv < kF32Keys ? nv : kF32Keys;
  };
  // K and V are read through buffer descriptors that end at the tile's last valid key: rows
  // past it read as zero, so what a page holds there never reaches a product.
  // K goes to LDS by DMA: an instruction moves 1 KB of whole rows, lane l the 16-byte
  // chunk that belongs at position l of it.  Chunk c of row r sits at position
  // c ^ (r mod 16) of its row, so that the operand reads (one chunk of 16 consecutive
  // rows a pass) touch every bank once.
  constexpr int CPR = D / 4, RPI = kWave / CPR;  // chunks per row, rows per instruction
  float* const k_lds = o_lds + wave * kF32Keys * D;
  auto load_k = [&](int64_t off, int nv) {
    const u32x4 rsrc = buffer_rsrc(kp + off, nv * D * 4);
    int at = (lane / CPR) * D * 4 + (((lane % CPR) ^ (lane / CPR)) << 4);
    uint32_t dst = lds_offset(k_lds);
    asm volatile("" : "+v"(at), "+s"(dst));  // form the instructions' offsets here, not in registers across the loop
#pragma unroll
    for (int m = 0; m < kF32Keys / RPI; ++m)
      dma_16x64(rsrc, (at ^ (((RPI * m) % 16) << 4)) + m * kWave * 16, dst + m * kWave * 16);
  };
  auto load_v = [&](int64_t off, int nv) {
    const u32x4 r = buffer_rsrc(vp + off, nv * D * 4);
    const auto rsrc =
        __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(static_cast<uint64_t>(r[1]) << 32 | r[0]), 0, r[2], r[3]);
    const int at = (4 * half * D + DT * col) * 4;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int from = at + (i % 4) * D * 4, group = 8 * (i / 4) * D * 4;
      if constexpr (DT == 4) vr[i] = __builtin_bit_cast(vdt, __builtin_amdgcn_raw_buffer_load_b128(rsrc, from, group, 0));
      else vr[i] = __builtin_bit_cast(vdt, __builtin_amdgcn_raw_buffer_load_b64(rsrc, from, group, 0));
    }
  };

  __builtin_amdgcn_s_waitcnt(vmcnt_only(0));  // Q has landed: no wait for it inside the loop
  for (int first = 0; first < count; first += NT) {
    const int ntiles =
        2 * __builtin_amdgcn_readfirstlane(decode_tiles<NT>(a, head_table(a, h), list, count, first, table, scan_tmp));
    // this wave's next tile with a valid key at or after t
    int64_t off = 0;
    auto seek = [&](int& t) -> int {
      for (; t < ntiles; t += NW) {
        const int nv = tile_of(t, off);
        if (nv > 0) return nv;
      }
      return 0;
    };
    int t = wave, nvalid = seek(t);
    if (nvalid > 0) {
      load_k(off, nvalid);
      load_v(off, nvalid);
    }
    while (nvalid > 0) {
      // K has landed when at most the 16 V loads issued after its DMA are outstanding
      asm volatile("s_waitcnt vmcnt(16)" ::: "memory");
      f32x16 s0 = f32x16{};
      int at = col * D * 4 + ((half ^ (col % 16)) << 4);  // chunk 2 u + half of row col: at ^ (u << 5)
      asm volatile("" : "+v"(at));
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const f32x4 k = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(k_lds) + (at ^ (u << 5)));
#pragma unroll
        for (int e = 0; e < 4; ++e) s0 = __builtin_amdgcn_mfma_f32_32x32x2f32(k[e], q[u][e], s0, 0, 0, 0);
      }
      t += NW;
      const int next_valid = seek(t);
      // V, in flight since the last PV run, has landed: said here, so that no later wait for it
      // counts the DMA issued next
      __builtin_amdgcn_s_waitcnt(vmcnt_only(0));
      if (next_valid > 0) load_k(off, next_valid);
      if (nvalid < kF32Keys) {  // the block's last tile: keys past its end count for nothing
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (8 * (i / 4) + 4 * half + i % 4 >= nvalid) s0[i] = -INFINITY;
      }
      float mx = s0[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s0[i]);
      mx = pair_max(mx) * a.scale;
      if (__any(mx > m_run)) {  // rescale only when some row's running max grows
        const float m_new = fmaxf(m_run, mx);
        const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run - m_new) * kLog2e);
        l_run *= alpha;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[dt][i] *= alpha;
        m_run = m_new;
      }
      const float m0 = m_run == -INFINITY ? 0.f : m_run;
      // scale * s - max with one rounding, before the change to log2 units: the exponent's
      // error is then relative to its distance from the max
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        s0[i] = __builtin_amdgcn_exp2f(fmaf(s0[i], a.scale, -m0) * kLog2e);
        sum += s0[i];
      }
      l_run += sum;
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[i][dt], s0[i], o[dt], 0, 0, 0);
      if (next_valid > 0) load_v(off, next_valid);
      nvalid = next_valid;
    }
    __syncthreads();  // every wave is done with the table
  }

  // ---- the waves' partial results meet in LDS: O^T element (dt, i) is d = DT c + dt of
  // c = 8 (i / 4) + 4 half + i % 4
  const float l_tot = pair_sum(l_run);
  if (half == 0) {
    m_lds[wave][col] = m_run;
    l_lds[wave][col] = l_tot;
  }
  float* mine = o_lds + (wave * kF32Rows + col) * STRIDE;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    vdt w;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) w[dt] = o[dt][i];
    *reinterpret_cast<vdt*>(mine + DT * (8 * (i / 4) + 4 * half + i % 4)) = w;
  }
  __syncthreads();
  constexpr int C4 = D / 4;  // 16-byte pieces per output row
  for (int i = tid; i < kF32Rows * C4; i += NT) {
    const int r = i / C4, c4 = i % C4, row = row0 + r;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = fmaxf(m, m_lds[w][r]);
    float l = 0.f;
    f32x4 acc = f32x4{};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float weight = m_lds[w][r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_lds[w][r] - m) * kLog2e);
      const f32x4 ow = *reinterpret_cast<const f32x4*>(o_lds + (w * kF32Rows + r) * STRIDE + 4 * c4);
      l = fmaf(weight, l_lds[w][r], l);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(weight, ow[e], acc[e]);
    }
    if (row < row_end) {
      const float inv = l > 0.f ? 1.0f / l : 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] *= inv;
      *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + (static_cast<int64_t>(row) * a.H + h) * D + 4 * c4) = acc;
      if (a.lse && c4 == 0) a.lse[static_cast<int64_t>(h) * a.lq + row] = l > 0.f ? m + logf(l) : -INFINITY;
    }
  }
}

constexpr int kMaxDevices = 64;

// The current device, or -1 where its cached values have no slot.
int current_device() {
  int dev = -1;
  return hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < kMaxDevices ? dev : -1;
}

// The current device's CUs, looked up once per device.
int device_cus() {
  static std::atomic<int> known[kMaxDevices];
  const int dev = current_device();
  int n = dev >= 0 ? known[dev].load(std::memory_order_relaxed) : 0;
  if (n <= 0) {
    if (dev < 0 || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
      n = 256;
    if (dev >= 0) known[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// Workgroups of the one-wave-per-group kernel: one wave per group, at most as many
// workgroups as the device holds at once (its CU count times the kernel's
// occupancy, looked up once per device).
template <int D>
int group_workgroups(int64_t groups) {
  static std::atomic<int> resident[kMaxDevices];
  const int dev = current_device();
  int n = dev >= 0 ? resident[dev].load(std::memory_order_relaxed) : 0;
  if (n <= 0) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_attn_bf16_groups<D>, kGrpWaves * kWave, 0) !=
            hipSuccess ||
        per_cu <= 0)
      per_cu = 1;
    n = device_cus() * per_cu;
    if (dev >= 0) resident[dev].store(n, std::memory_order_relaxed);
  }
  const int64_t need = (groups + kGrpWaves - 1) / kGrpWaves;
  return static_cast<int>(need < n ? need : n);
}

}  // namespace

hipError_t launch_attention(const CacheGeom& g, const AttnLaunch& L, hipStream_t stream) {
  AttnArgs a;
  a.q = L.q;
  a.k_pages = g.k_pages;
  a.v_pages = g.v_pages;
  a.page_table = g.page_table;
  a.pt_stride = g.pt_stride;
  a.num_pages = g.num_pages;
  a.H = g.H;
  a.S = g.S;
  a.B = g.B;
  a.Bpc = g.Bpc;
  a.nb = g.nb;
  a.lq = L.lq;
  a.G = L.group_size;
  a.R = L.R;
  a.idx = L.idx;
  a.cnt = L.cnt;
  a.top_k = L.top_k;
  a.dense_first = L.dense_first_block;
  a.dense_count = L.dense_num_blocks;
  a.scale = L.scale;
  a.out = L.out;
  a.lse = L.lse;
  a.first_wg = 0;
  const int rows = L.group_size < L.lq ? L.group_size : L.lq;
  const int64_t groups = static_cast<int64_t>(g.H) * L.R;
  if (groups <= 0 || groups > 0x7fffffff) return groups <= 0 ? hipSuccess : hipErrorInvalidConfiguration;
  auto launch = [&](auto kernel, int rows_per_wg, int threads) {
    a.tiles_per_group = (rows + rows_per_wg - 1) / rows_per_wg;
    const int64_t nwg = groups * a.tiles_per_group;
    if (nwg > 0x7fffffff) return hipErrorInvalidConfiguration;
    return launch_kernel(kernel, dim3(static_cast<unsigned>(nwg)), dim3(threads), 0, stream, a);
  };
  // A group of one row has a workgroup of its own, and a grid holds fewer than 2^32 threads,
  // 8.4 M workgroups at d = 64: more of them go in several grids.
  auto launch_f32 = [&](auto kernel, int threads) {
    a.tiles_per_group = (rows + kF32Rows - 1) / kF32Rows;
    const int64_t nwg = groups * a.tiles_per_group, most = 0xffffffffll / threads;
    if (nwg > 0x7fffffff) return hipErrorInvalidConfiguration;
    LaunchStatus st;
    for (int64_t first = 0; first < nwg; first += most) {
      a.first_wg = static_cast<int>(first);
      st(kernel, dim3(static_cast<unsigned>(nwg - first < most ? nwg - first : most)), dim3(threads), 0, stream, a);
    }
    return st.err;
  };
  if (g.dtype != 0) {
    if (g.D == 128) return launch_f32(k_attn_f32<128>, F32Shape<128>::NW * kWave);
    return launch_f32(k_attn_f32<64>, F32Shape<64>::NW * kWave);
  }
  if (rows <= 32) {  // one 32-row tile per group: a wave per group
    a.tiles_per_group = 1;
    const dim3 threads(kGrpWaves * kWave);
    if (g.D == 128)
      return launch_kernel(k_attn_bf16_groups<128>, dim3(group_workgroups<128>(groups)), threads, 0, stream, a);
    return launch_kernel(k_attn_bf16_groups<64>, dim3(group_workgroups<64>(groups)), threads, 0, stream, a);
  }
  constexpr int kThreads = kR64Waves * kWave, kRows = kR64Waves * 64;
  static_assert(kRows == kAttnRows && kR32Waves * 32 == kAttnRows, "rows of a workgroup with one key stream");
  // the longest list that a group may have, in tiles
  const int64_t blocks = L.idx == nullptr ? L.dense_num_blocks : L.top_k < g.nb ? L.top_k : g.nb;
  const int streams = attn_key_streams(g.D, groups, rows, blocks * (g.B / kTileKeys), device_cus());
  if (g.D == 128) {
    if (streams == 2) return launch(k_attn_bf16_r64<2>, kRows / 2, kThreads);
    return launch(k_attn_bf16_r64<1>, kRows, kThreads);
  }
  switch (streams) {
    case 4: return launch(k_attn_bf16_r32<4>, kRows / 4, kR32Waves * kWave);
    case 2: return launch(k_attn_bf16_r32<2>, kRows / 2, kR32Waves * kWave);
    default: return launch(k_attn_bf16_r32<1>, kRows, kR32Waves * kWave);
  }
}

}  // namespace omnimem
