// For each line "M N K block cus" of the standard input, the plan of the
// dequantise-on-load GEMM: its kernel in words (no spaces), row tiles, column tiles
// or weight-row groups, ranges of K, workgroups, modelled us, and the measure of its
// sums' error with the limit that the plan has to keep.
#include <cstdint>
#include <cstdio>
#include <string>

#include "zq_gemm_plan.h"

using namespace zq;

int main() {
  long long M, N, K, block, cus;
  while (std::scanf("%lld %lld %lld %lld %lld", &M, &N, &K, &block, &cus) == 5) {
    int lg = 0;
    while ((1 << lg) < block) ++lg;
    const GemmPlan p = gemm_plan(M, N, K, lg, cus);
    std::string name;
    double drift = 0.0, limit = 0.0;
    const std::string split = p.splits > 1 ? ",split" : "";
    if (p.route == GemmRoute::kRows) {
      const RowsVariant& v = kRowsVariants[p.kind];
      name = (v.ks ? "ranges:" : "rows:") + std::to_string(v.mt) + "x" + std::to_string(v.ng) + ",waves" +
             std::to_string(v.w) + (v.xl ? ",staged" : "") + (v.sets > 1 ? ",sets" + std::to_string(v.sets) : "");
      drift = sum_drift((double)K / (double)(p.splits * v.w * v.sets), p.splits > 1 ? (double)p.splits : 0.0, v.w);
    } else if (p.route == GemmRoute::kGemv) {
      name = "stream:" + std::to_string(p.kc) + split;
      drift = sum_drift((double)(p.kc < K ? p.kc : K), (double)p.splits, 0.0);
    } else if (p.route == GemmRoute::kTiles) {
      const TileShape& t = kTileShapes[p.kind];
      name = "tiles:" + std::to_string(t.bm) + "x" + std::to_string(t.bn) + split;
      drift = sum_drift((double)(ceil_div(K / kGemmKStep, p.splits) * kGemmKStep) / t.sets, (double)p.splits, 0.0);
    } else {
      name = "plain";
    }
    if (M <= kGemvRows) {
      const int64_t kc = gemv_range(N, K);
      limit = kDriftSlack * sum_drift((double)(kc < K ? kc : K), K > kc ? (double)ceil_div(K, kc) : 1.0, 0.0);
    } else {
      limit = drift_limit(M, N, k_splits(K), cus);
    }
    std::printf("%s %lld %lld %lld %lld %.4f %.1f %.1f\n", name.c_str(), (long long)p.mtiles, (long long)p.ntiles,
                (long long)p.splits, (long long)p.grid, p.us, drift, limit);
  }
  return 0;
}
