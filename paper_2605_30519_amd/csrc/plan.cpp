// plan.cpp -- workspace plans of the selection and the union-gather comparator
// (host only).
#include "plan.h"

namespace omnimem {

SelectPlan plan_select(const CacheGeom& g, int lq, int K, int G, int E, float scale, int awe, int score_mode) {
  SelectPlan p{};
  p.score_mode = score_mode;
  p.lq = lq;
  p.G = G;
  p.R = (lq + G - 1) / G;
  p.K = K;
  p.awe = awe;
  p.first_excluded = awe ? (g.n - E) * g.Bpc : g.nb;
  p.scale = scale;
  const int rows = G < lq ? G : lq;
  p.qsplit = (rows + kQRowsPerSplit - 1) / kQRowsPerSplit;
  p.inline_scores = p.R <= kInlineGroups;
  size_t off = 0;
  p.off_qpart = off;
  off = align256(off + static_cast<size_t>(g.H) * p.R * p.qsplit * g.D * sizeof(float));
  p.off_kbar = off;
  if (!p.inline_scores) off = align256(off + static_cast<size_t>(g.H) * g.nb * g.D * sizeof(float));
  p.off_keys = off;
  off = align256(off + static_cast<size_t>(g.H) * p.R * ((g.nb + 3) / 4 * 4 + (g.nb == 0)) * sizeof(uint32_t));
  p.off_part = off;
  if (score_mode == 1) {
    constexpr int kSliceRows = kProbSliceRows;
    p.prob_multi = G <= kSliceRows / 2;
    if (p.prob_multi) {
      p.prob_gps = kSliceRows / G;
      p.prob_spg = 1;
      p.prob_slices = (p.R + p.prob_gps - 1) / p.prob_gps;
      p.prob_nseg = p.R;
    } else {
      p.prob_gps = 1;
      p.prob_spg = (rows + kSliceRows - 1) / kSliceRows;
      p.prob_slices = p.R * p.prob_spg;
      p.prob_nseg = p.prob_slices;
    }
    if (!p.prob_multi) off = align256(off + static_cast<size_t>(g.H) * p.prob_nseg * g.nb * sizeof(float));
    p.off_ksplit = off;
    off = align256(off + static_cast<size_t>(g.H) * ((g.nb + 63) / 64) * 2 * 64 * g.D * sizeof(uint16_t));
  }
  p.total = off;
  return p;
}

// A workgroup of KS streams takes 256 / KS rows and every KS-th tile of its list, and a CU
// runs one workgroup at a time, so the time goes as the rounds of workgroups over CUs times
// (what a workgroup's start and end take + its tiles).  The costs, in 10 ns, are fitted to
// 98 timings of each kernel and stream count on 256 CUs: 2 to 40 heads, groups of 64 to 4,680
// rows, 1 to 64 tiles.  A choice by rounds and 1 / KS alone, as for lists of 64 tiles, took
// up to 3.3 times the best time (d = 64, 40 heads x 3 groups x 1,560 rows, 1 tile: 78 us with
// four streams, 24 with one); this one is within 8% of the best of them everywhere, on average
// 0.2%.  Some of them, in us with 1 / 2 / 4 streams:
//   d = 128: 5 heads x 3 x 1,560 rows, 64 tiles 98 / 60, 1 tile 12.6 / 13.5;
//            40 x 3 x 1,560, 8 tiles 86 / 109, 64 tiles 416 / 429; 12 x 4,680, 64: 111 / 123
//   d = 64:  16 x 1,560, 64 tiles 82 / 44 / 53, 1 tile 7.4 / 8.3 / 14.6;
//            40 x 1,560, 4 tiles 18 / 20 / 26, 64 tiles 139 / 128 / 106
int attn_key_streams(int D, int64_t groups, int rows, int64_t tiles, int cus) {
  struct Cost {
    int start, tile;
  };
  static constexpr Cost k128[] = {{907, 139}, {934, 153}}, k64[] = {{347, 108}, {437, 115}, {497, 128}};
  const Cost* cost = D == 128 ? k128 : k64;
  int best = 1;
  double least = 0;
  for (int ks = 1; ks <= (D == 128 ? 2 : 4); ks *= 2, ++cost) {
    const int per_wg = kAttnRows / ks;
    const int64_t rounds = (groups * ((rows + per_wg - 1) / per_wg) + cus - 1) / cus;
    const double tiles_time = static_cast<double>(cost->tile) * static_cast<double>((tiles + ks - 1) / ks);
    const double time = static_cast<double>(rounds) * (cost->start + tiles_time);
    if (ks == 1 || time < least) {
      best = ks;
      least = time;
    }
  }
  return best;
}

UnionPlan plan_union(const CacheGeom& g) {
  UnionPlan u{};
  const size_t eb = g.dtype == 0 ? 2 : 4;
  u.slab_bytes = static_cast<int64_t>(g.B) * g.D * eb;
  const size_t nb = g.nb > 0 ? g.nb : 1;
  size_t off = 0;
  u.off_flags = off;
  off = align256(off + nb * sizeof(int32_t));
  u.off_table = off;
  off = align256(off + nb * sizeof(int32_t));
  u.off_kbuf = off;
  off = align256(off + nb * g.H * static_cast<size_t>(u.slab_bytes));
  u.off_vbuf = off;
  off = align256(off + nb * g.H * static_cast<size_t>(u.slab_bytes));
  u.total = off;
  return u;
}

}  // namespace omnimem
