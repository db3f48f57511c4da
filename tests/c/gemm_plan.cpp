// For each line "M N K block cus" of the standard input, the plan of the
// dequantise-on-load GEMM: its kernel in words (no spaces), row tiles, column tiles
// or weight-row groups, ranges of K, workgroups, modelled us.
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
    const std::string split = p.splits > 1 ? ",split" : "";
    if (p.route == GemmRoute::kRows) {
      const RowsVariant& v = kRowsVariants[p.kind];
      name = (v.ks ? "ranges:" : "rows:") + std::to_string(v.mt) + "x" + std::to_string(v.ng) + ",waves" +
             std::to_string(v.w) + (v.xl ? ",staged" : "");
    } else if (p.route == GemmRoute::kGemv) {
      name = "stream:" + std::to_string(p.kc) + split;
    } else if (p.route == GemmRoute::kTiles) {
      const TileShape& t = kTileShapes[p.kind];
      name = "tiles:" + std::to_string(t.bm) + "x" + std::to_string(t.bn) + split;
    } else {
      name = "plain";
    }
    std::printf("%s %lld %lld %lld %lld %.4f\n", name.c_str(), (long long)p.mtiles, (long long)p.ntiles,
                (long long)p.splits, (long long)p.grid, p.us);
  }
  return 0;
}
