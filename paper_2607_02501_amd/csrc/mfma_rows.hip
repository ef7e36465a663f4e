// mfma_rows.hip -- host side of the small-m matrix-core path (Q8_0 and Q4_0; paper section 3.2, backend-specific dispatch): the choice of tile
// and split of k for a lone projection, the tile of a fused run, and the
// dispatch to the kernels (mfma_rows.h).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "eb_internal.h"

namespace eb {

namespace {

// Workgroups of a tile that share a CU (LDS, and registers where NT = 4).
int per_cu(const RowsTiles &t) {
  constexpr int k8[3][4] = {{4, 2, 1, 1}, {3, 2, 1, 1}, {2, 1, 1, 1}}, k4[4] = {4, 3, 2, 2};
  return t.w == 4 ? k4[t.mb - 1] : k8[t.nt == 1 ? 0 : t.nt == 2 ? 1 : 2][t.mb - 1];
}

// Estimated time (us) of a lone launch: the launch and its first copies, then
// rounds of as many workgroups side by side as a CU takes.  In a round each
// workgroup's step of k (one block per wave) keeps the CU busy for the rows of
// x, the weight rows and their product, and waits for a while on its own; its
// ends (adding up the waves' tiles, the outputs) pass partly beside the others'.
// At least the time of reading x and the weights.  A split adds the reduction:
// its launch, its chain of loads and its traffic.
// Fitted to 56 thousand launches of 3200 problems (2 to 2500 rows, 16 to 26000
// outputs, k of 32 to 12288, both formats and activation types): 7% rms near the
// best tile, whose time the chosen tile's exceeds by 0.5% in the mean (up to 128
// rows and 6000 outputs), 1.2% (more outputs) and 2.4% (more rows).
// (tiles: workgroups of a split; per: its steps.)
double lone_us(const RowsTiles &t, uint32_t tiles, uint32_t per, double bytes, double outputs, uint32_t cus) {
  const double busy = t.w == 8 ? 0.076 * t.mb + 0.08 * t.nt + 0.021 * t.nt * t.mb : 0.22 + 0.056 * t.mb;
  const double step = busy + (t.w == 8 ? 0.065 : 0.125);
  const double ends = (t.w == 8 ? 1.1 : 0.22) + 0.057 * t.nt * t.mb * (t.w == 8 ? 1 : 2);
  auto round = [&](double c, double ends_c) {  // c workgroups per CU
    return ends * (0.67 + 0.33 * ends_c) + per * std::max(step, c * busy);
  };
  const uint32_t occ = (uint32_t)per_cu(t), units = tiles * (uint32_t)t.splits, full = units / (occ * cus);
  const uint32_t rest = units - full * occ * cus;
  double us = full ? full * round(occ, occ) : 0.0;
  if (rest > cus) {
    const double c = (rest + cus - 1) / cus;
    us += round(c, c);
  } else if (rest) {  // on a part of the CUs
    us += round(1, (double)rest / cus);
  }
  us = 2.7 + std::max(us, bytes / 3.85e6);
  if (t.splits > 1) us += 1.7 + 0.15 * t.splits + (t.splits + 1) * outputs * 4 / 2.86e6;
  return us;
}

}  // namespace

bool rows_fits(int64_t m, int64_t n, int64_t k) {
  // Above 128 rows the large-m tile kernel has the higher rate, but needs
  // more work to reach it (measured, Q8_0, us, this kernel against it: 160
  // rows 2048 -> 2560 9 against 18, 300 rows 1024 -> 1024 6 against 13, 816
  // rows 2048 -> 2560, 8.6 GFLOP, 25 against 30; 2000 rows 2976 -> 1000, 11.9
  // GFLOP, 32 against 30; 990 problems of 129 to 2500 rows up to 9 GFLOP 0.64
  // times as long in the mean).  Behind it are short k with outputs of 6 MB and
  // more, where a workgroup's ends count (2408 rows 64 -> 5685 27 against 22):
  // they stay here for the exact weights.  Offsets inside a tile's rows of x,
  // weights and y stay below 2^31 (an offset of 2^31 or more reads zero and
  // stores nothing).
  return m >= 1 && (m <= kRowsMaxM || 2.0 * (double)m * (double)n * (double)k <= kRowsMaxFlops) &&
         64 * k * 2 < 0x7fff0000LL && 64 * n * 4 < 0x7fff0000LL;
}

RowsTiles rows_plan(int32_t type, int64_t m, int64_t n, int64_t k, size_t max_ws, int cus, bool norm_next) {
  const int steps = (int)((k / kQK + 7) / 8), most = std::max(1, std::min(kRowsMaxSplits, steps));
  // Few columns (16-row tiles of the weights for a third of the CUs at most): from
  // k = 4096 on a split takes less than the estimate says (0.75 times as long as
  // unsplit in the mean of 123 problems of 2 to 128 rows; equal at 2048 to 4095,
  // 1.2 to 1.4 times below), and a reduction may save the row kernel.
  const bool few = m <= kRowsMaxM && cus / ((n + 15) / 16) >= 3;
  const double unsplit_us = few && (norm_next || k >= 4096) ? kNormLaunchUs : 0.0;
  const double bytes = 2.0 * m * k + (double)n * k * (type == EB_Q8_0 ? 34 : 18) / 32;
  const int64_t stride = (m * n + 63) / 64 * 64;
  const uint32_t blocks = (uint32_t)(k / kQK);
  RowsTiles best;
  double best_t = 0;
  for (int c = 0; c < 4; ++c)  // weight rows and waves: 16, 32 and 64 with eight, 64 with four
    for (int mb = 1; mb <= 4; ++mb) {
      if (mb > 1 && 16 * (mb - 1) >= m) continue;
      RowsTiles t;
      t.nt = c < 3 ? 1 << c : 4;
      t.mb = mb;
      t.w = c < 3 ? 8 : 4;
      const uint32_t tiles = (uint32_t)rows_units(t, m, n), all = (blocks + t.w - 1) / t.w;
      for (int sp = 1; sp <= most; ++sp) {
        if (sp > 1 && (size_t)(stride * sp * 4) > max_ws) break;
        if (sp > 1 && (steps + sp - 1) / sp == (steps + sp - 2) / (sp - 1)) continue;  // no shorter
        t.splits = sp;
        t.ws_stride = sp > 1 ? stride : 0;
        double us = lone_us(t, tiles, (all + sp - 1) / sp, bytes, (double)(m * n), cus) + (sp == 1 ? unsplit_us : 0.0);
        // Between estimates that differ by less than their error: 32-row tiles of
        // the weights for one row block and many outputs (the chosen tile's time
        // then exceeds the best one's by 0.9% instead of 1.25%, 457 problems),
        // higher tiles for more rows (0.6% instead of 0.8%).
        if (m <= 16 ? n > 4096 && t.nt != 2 : mb == 1) us *= m <= 16 ? 1.05 : 1.035;
        if (best.nt == 0 || us < best_t) {
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
