// mfma_rows.hip -- host side of the small-m matrix-core path (Q8_0 and Q4_0; paper section 3.2, backend-specific dispatch): the choice of tile
// and split of k for a lone projection, the tile of a fused run, and the
// dispatch to the kernels (mfma_rows.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "eb_internal.h"

namespace eb {

namespace {

// Estimated time (us) of a lone launch: a launch and its first copies, then
// for every round of workgroups over the CUs its steps of k (one block per
// wave), each with a part for the rows of x, for the weight rows and for their
// product.  Most tiles of eight waves have a CU to themselves; of those of four
// (NT = 4) two share one, and of those of at most 16 rows and 32 weight rows
// three or more, which then take turns at 0.85 of a round each without the last
// one's idle CUs (Q8_0 11008 x 4096 at 2 to 16 rows: 64-row tiles of the weights
// 14.0 to 15.2 us, 32-row ones 12.8 to 13.8).  Fitted to launches of 1024..4096 -> 1024..8192 at
// 16 to 816 rows (Q8_0, bfloat16): within 15%, and it ranks the tiles as the
// measurements do.
double lone_us(const RowsTiles &t, int64_t m, int64_t n, int64_t k, int cus) {
  const int64_t units = ((n + 16 * t.nt - 1) / (16 * t.nt)) * ((m + 16 * t.mb - 1) / (16 * t.mb)) * t.splits;
  const int64_t steps = (k / kQK + t.w - 1) / t.w, per = (steps + t.splits - 1) / t.splits;
  double us = 3.0;
  if (t.w == 8) {
    const double step = 0.115 + 0.05 * t.mb + 0.105 * t.nt + 0.02 * t.nt * t.mb;
    double rounds = (double)((units + cus - 1) / cus);
    if (t.mb == 1 && t.nt <= 2) rounds = std::max(1.0, 0.85 * (double)units / cus);
    us += rounds * (double)per * step;
  } else {
    const int64_t rounds = (units + 2 * cus - 1) / (2 * cus);
    const double step = (0.3 + 0.17 * t.mb) * (units <= cus ? 0.7 : 1.0);
    us += (rounds > 1 ? 0.85 : 1.0) * (double)rounds * (double)per * step;
  }
  // the reduction of the partial sums: a launch, and their traffic
  if (t.splits > 1) us += 3.2 + (double)(t.splits + 1) * (double)m * (double)n * 4 / 4e6;
  return us;
}

}  // namespace

bool rows_fits(int64_t m, int64_t n, int64_t k) {
  // Above 128 rows the large-m tile kernel has the higher rate, but needs
  // more work to reach it (measured, Q8_0, us, this kernel against it: 160
  // rows 2048 -> 2560 9 against 18, 300 rows 1024 -> 1024 6 against 13, 816
  // rows 2048 -> 2560, 8.6 GFLOP, 25 against 30; 2000 rows 2976 -> 1000, 11.9
  // GFLOP, 32 against 30).  Offsets inside a tile's rows of x, weights and y stay below
  // 2^31 (an offset of 2^31 or more reads zero and stores nothing).
  return m >= 1 && (m <= kRowsMaxM || 2.0 * (double)m * (double)n * (double)k <= kRowsMaxFlops) &&
         64 * k * 2 < 0x7fff0000LL && 64 * n * 4 < 0x7fff0000LL;
}

RowsTiles rows_plan(int64_t m, int64_t n, int64_t k, size_t max_ws, int cus) {
  // When the 16-row tiles of the weights leave two thirds of the CUs idle, k
  // is split whatever the estimate says: in a layer chain the reduction then
  // also normalises for the next projection, a launch that would follow anyway.
  const int64_t wgs = (n + 15) / 16, steps = (k / kQK + 7) / 8;
  const int most = (int)std::max<int64_t>(1, std::min<int64_t>(kRowsMaxSplits, steps));
  const bool split = m <= kRowsMaxM && cus / wgs >= 3 && most > 1;
  RowsTiles best;
  double best_t = 0;
  for (int sp = 1; sp <= most; ++sp) {
    const int64_t stride = (m * n + 63) / 64 * 64;
    if (sp > 1 && (size_t)(stride * sp * 4) > max_ws) break;
    if (sp > 1 && (steps + sp - 1) / sp == (steps + sp - 2) / (sp - 1)) continue;  // no shorter
    for (int c = 0; c < 4; ++c)  // weight rows and waves: 16, 32 and 64 with eight, 64 with four
      for (int mb = 1; mb <= 4; ++mb) {
        if (mb > 1 && 16 * (mb - 1) >= m) continue;
        RowsTiles t;
        t.nt = c < 3 ? 1 << c : 4;
        t.mb = mb;
        t.w = c < 3 ? 8 : 4;
        t.splits = sp;
        t.ws_stride = sp > 1 ? stride : 0;
        const double us = lone_us(t, m, n, k, cus);
        if (best.nt == 0 || (split && best.splits == 1 && sp > 1) || us < best_t) {
          best_t = us;
          best = t;
        }
      }
  }
  return best;
}

int64_t rows_units(const RowsTiles &t, int64_t m, int64_t n) {
  return ((n + 16 * t.nt - 1) / (16 * t.nt)) * ((m + 16 * t.mb - 1) / (16 * t.mb));
}

RowsTiles rows_plan_multi(const std::vector<MMOp> &ops, int cus) {
  int max_m = 1;
  for (const MMOp &o : ops) max_m = std::max(max_m, (int)o.m);
  // the fewest row tiles of at most 64 rows, evenly high; the widest weight
  // tile that still gives every CU a workgroup (wider ones read x less often)
  RowsTiles t;
  const int blocks = (max_m + 15) / 16, tiles_m = (blocks + 3) / 4;
  t.mb = (blocks + tiles_m - 1) / tiles_m;
  for (t.nt = 4; t.nt > 1; t.nt /= 2) {
    int64_t units = 0;
    for (const MMOp &o : ops) units += rows_units(t, o.m, o.n);
    if (units >= cus) break;
  }
  t.w = t.nt == 4 ? 4 : 8;
  return t;
}

hipError_t launch_rows(int32_t type, int32_t xt, const RowsTiles &t, const MMOp &o, float *ws,
                       hipStream_t s) {
  if (!rows_fits(o.m, o.n, o.k) || (t.splits > 1 && !ws)) return hipErrorInvalidValue;
  float *part = t.splits > 1 ? ws : nullptr;
  if (type == EB_Q4_0) return rows_lone<EB_Q4_0>(xt, t, o, t.splits, part, t.ws_stride, s);
  return rows_lone<EB_Q8_0>(xt, t, o, t.splits, part, t.ws_stride, s);
}

hipError_t launch_rows_multi(int32_t type, int32_t xt, const RowsTiles &t, const MMOp *dev_ops,
                             int nops, int64_t units, hipStream_t s) {
  if (nops < 1 || units < 1 || units > 0x7fffffff) return hipErrorInvalidValue;
  if (type == EB_Q4_0) return rows_multi<EB_Q4_0>(xt, t, dev_ops, nops, units, s);
  return rows_multi<EB_Q8_0>(xt, t, dev_ops, nops, units, s);
}

MMOp rows_op(int32_t type, const void *w, int64_t n, int64_t k, const void *x, int64_t m, void *y,
             int32_t yt, const Fuse &f) {
  const Layout L = layout_of(type, n, k);
  MMOp e{};
  e.w = static_cast<const uint8_t *>(w);
  e.x = static_cast<const uint16_t *>(x);
  e.y = y;
  e.d_off = L.d_off;
  e.ds = (int32_t)L.ds;
  e.m = (int32_t)m;
  e.n = (int32_t)n;
  e.k = (int32_t)k;
  e.yt = yt;
  e.f = f;
  return e;
}

}  // namespace eb
