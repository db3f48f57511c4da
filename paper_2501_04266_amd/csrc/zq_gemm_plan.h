// zq_gemm_plan.h -- which kernel of the dequantise-on-load GEMM runs a product,
// in which tiles and splits: host arithmetic on the sizes and the number of CUs
// alone, without HIP, so that a test on the CPU can ask it.
#pragma once

#include <stdint.h>

namespace zq {

constexpr int kGemmKStep = 64;                        // K is a multiple of this
constexpr int64_t kGemmPpMaxK = int64_t(1) << 21;     // 32-bit buffer offsets in the ping-pong kernel
constexpr int64_t kGemmMaxSplits = 16;                // K splits of the ping-pong kernel's tiles
constexpr int64_t kGemmHalfM = 128;                   // rows up to which its tiles have 128 rows
// one atomic addition into y with the GPU's others (measured: about 330 G/s), us
constexpr double kGemmAtomicUs = 3e-6;
constexpr int64_t kGemvRows = 16;                     // k_dqgemv: rows of x
constexpr int64_t kGemvKc = 1024;                     // its longest K range
constexpr int64_t kGemvTargetWgs = 1024;              // workgroups it aims at
constexpr int64_t kScaleLds = 8192;                   // k_dqrows: scales a workgroup can stage,
constexpr int64_t kRangeScales = 64;                  // of them a row's, where K is split over the grid,
constexpr int64_t kXLds = 49152;                      // and bytes of x
constexpr int64_t kRowsXcds = 8;

// k_dqrows' variants: row tiles and weight-row tiles of 16 a workgroup, waves, steps
// loaded ahead, x staged in LDS, K split over the grid, accumulator sets.  Two sets
// cost nothing where memory binds or their registers leave as many workgroups on a
// CU; else there is a variant of one set too (64 rows, N = K = 2048: 9.0 us with one
// set, 9.3 with two; 260 rows, N = 6144, K = 2048 in 4 x 4 tiles: 22.3 and 28.4, since
// one workgroup of them fills a CU's registers and two of the other).
struct RowsVariant {
  int mt, ng, w, d;
  bool xl, ks;
  int sets;
};
constexpr RowsVariant kRowsVariants[] = {
    {1, 3, 8, 2, true, false, 2},   {1, 1, 8, 6, true, false, 2},  {1, 6, 8, 2, false, false, 1},
    {1, 5, 8, 3, false, false, 1},  {1, 4, 8, 2, false, false, 1}, {1, 3, 8, 3, false, false, 1},
    {1, 2, 16, 2, false, false, 2}, {2, 6, 8, 2, false, false, 2}, {2, 5, 8, 2, false, false, 2},
    {2, 4, 8, 2, false, false, 2},  {2, 3, 8, 2, false, false, 2}, {2, 2, 8, 2, false, false, 1},
    {2, 2, 8, 2, false, false, 2},  {4, 2, 8, 2, false, false, 1}, {4, 2, 8, 2, false, false, 2},
    {4, 2, 4, 2, false, false, 1},  {4, 2, 4, 2, false, false, 2}, {4, 3, 4, 2, false, false, 1},
    {4, 3, 4, 2, false, false, 2},  {4, 4, 4, 2, false, false, 1}, {4, 4, 4, 2, false, false, 2},
    {4, 5, 4, 2, false, false, 2},  {4, 6, 4, 1, false, false, 2}, {1, 6, 8, 2, false, true, 2},
    {2, 6, 8, 2, false, true, 2},
};
constexpr int kRowsKinds = sizeof(kRowsVariants) / sizeof(kRowsVariants[0]);

// The ping-pong kernel's tile shapes: rows and columns of y, accumulator sets, and
// the time of one 64-wide K-step of a tile with few CUs busy and with all of them
// (measured over the layers' GEMMs: 256 x 256 1.2 us in a round of an eighth to a
// quarter of the CUs, 1.3-1.5 in half to three quarters, 1.75 in full ones; 256 x 192
// 1.15, 1.28 and 1.40-1.48; 256 x 128 0.85, 0.95-1.0 and 1.0-1.14).
struct TileShape {
  int bm, bn, sets;
  double step0_us, step1_us;
};
constexpr TileShape kTileShapes[] = {
    {128, 256, 2, 0.9, 0.9}, {256, 256, 1, 1.0, 1.75}, {256, 192, 1, 0.78, 1.46}, {256, 128, 2, 0.85, 1.05}};

enum class GemmRoute { kRows, kGemv, kTiles, kPlain };
struct GemmPlan {
  GemmRoute route;
  int kind;                         // of kRowsVariants or kTileShapes
  int64_t mtiles, ntiles, splits;   // row tiles, column tiles (weight-row groups), ranges of K
  int64_t grid;                     // workgroups
  int64_t kc;                       // k_dqgemv: K per range
  double us;                        // modelled time
};

// What a sum's error grows with: its square is close to proportional to the length
// K of one accumulator's chain of MFMA additions, plus 8 for each range of K added up
// in y and 4 for each wave's part added up in LDS (measured against 64 bits, K 960
// to 28672, every kernel: the 2-norm of the error is 6e-9 times the root of that,
// within a tenth).
inline double sum_drift(double k_chain, double ranges, double waves) { return k_chain + 8.0 * ranges + 4.0 * waves; }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// the same of counts below 2^53, as a double: a plan takes some hundred of these, and
// a 64-bit integer division is the longest instruction there is (0.3 us a plan)
inline double ceil_ratio(int64_t a, int64_t b) {
  const double q = (double)(int64_t)((double)a / (double)b);
  return q * (double)b < (double)a ? q + 1.0 : q;
}

// K-steps of the longest range where K is split s ways
struct KSplits {
  int64_t most;
  double steps[kGemmMaxSplits + 1];
};
inline KSplits k_splits(int64_t K) {
  KSplits k;
  const int64_t ksteps = K / kGemmKStep;
  k.most = ksteps < 1 ? 1 : ksteps < kGemmMaxSplits ? ksteps : kGemmMaxSplits;
  for (int64_t s = 1; s <= k.most; ++s) k.steps[s] = ceil_ratio(ksteps, s);
  return k;
}

// k_dqgemv's K range: halved (down to 256) until about kGemvTargetWgs workgroups run
inline int64_t gemv_range(int64_t N, int64_t K) {
  int64_t kc = kGemvKc;
  while (kc > 256 && ceil_div(N, 64) * ceil_div(K, kc) < kGemvTargetWgs) kc /= 2;
  return kc;
}

// The drift that no plan exceeds (kDriftSlack: by more than a fortieth of the error).
// Up to 16 rows that of k_dqgemv, beyond that of 256 x 256 tiles (128 x 256 up to
// 128 rows) with one set of accumulators, split until they fill rounds of CUs at the
// price of the additions into y: a faster plan that sums longer chains than these is
// not taken (256 rows, N = 18432, K = 6144 in 256 x 192 tiles of whole K: 108 us and
// an error of 4.9e-7, where tiles of K split three ways have 2.7e-7).
constexpr double kDriftSlack = 1.05;
inline double drift_limit(int64_t M, int64_t N, const KSplits& ks, int64_t cus) {
  const bool half = M <= kGemmHalfM;
  const int64_t tiles = ceil_div(M, half ? 128 : 256) * ceil_div(N, 256);
  const double step = half ? 0.9 : 1.5, added = (double)M * (double)N * kGemmAtomicUs;
  int64_t best = 1;
  double best_us = 0.0;
  for (int64_t s = 1; s <= ks.most; ++s) {
    const double us = ceil_ratio(tiles * s, cus) * ks.steps[s] * step + (s > 1 ? (double)s * added : 0.0);
    if (s == 1 || us < best_us) {
      best = s;
      best_us = us;
    }
  }
  return kDriftSlack * sum_drift(ks.steps[best] * kGemmKStep, (double)best, 0.0);
}

// K splits of the ping-pong kernel's tiles, and the modelled time in us (negative:
// every count exceeds the drift limit).  A tile's workgroup fills a CU (its LDS
// buffers alone take 110-147 KB), so the tiles run in rounds of one workgroup per
// CU, and a last round that is mostly empty idles much of the GPU (72 tiles on 256
// CUs use 28% of it).  Splitting K s ways makes s times as many workgroups of 1/s
// the K-steps, at the price of a zero fill of y and M N s atomic additions; the
// count taken minimises
//   (full rounds step1 + [a part of one] (step0 + (step1 - step0) part)) ceil(ksteps / s)
//   + 4, or 9.5 with the fill's launch, + [s > 1] M N s atomic (1/2 + 1/2 CUs / workgroups)
// where a K-step takes longer the more CUs run (the clock falls under load), and
// the additions of all rounds but the last overlap the next one's work.  It splits
// the GEMMs of a few hundred rows 2-16 ways and leaves full rounds whole.
inline int64_t tile_splits(int64_t tiles, const KSplits& ks, int64_t M, int64_t N, int64_t cus, const TileShape& t,
                           double load, double limit, double* us) {
  const double step0 = load * t.step0_us, step1 = load * t.step1_us, added = (double)M * (double)N * kGemmAtomicUs;
  int64_t best = 1;
  *us = -1.0;
  for (int64_t s = 1; s <= ks.most; ++s) {
    const double steps = ks.steps[s];
    if (sum_drift(steps * kGemmKStep / t.sets, (double)s, 0.0) > limit) continue;
    const double wgs = (double)(tiles * s), rnds = wgs / (double)cus, full = (double)(int64_t)rnds, part = rnds - full;
    const double rounds = full * step1 + (part > 0.0 ? step0 + (step1 - step0) * part : 0.0);
    const double alone = full > 0.0 ? (double)cus / wgs : 1.0;
    const double c = rounds * steps + (s > 1 ? (double)s * added * (0.5 + 0.5 * alone) + 9.5 : 4.0);
    if (*us < 0.0 || c < *us) {
      best = s;
      *us = c;
    }
  }
  return best;
}

// The ping-pong kernel's tile shape and K splits for a product, and its modelled
// time.  Up to 128 rows 128 x 256 tiles; beyond, the shape of 256 rows whose rounds
// of one tile per CU (with its best split) take the least: narrower tiles cost more
// per column, but where 256 columns leave a round part empty they fill it (1,024
// rows, QKV of the 6144-wide layer: 288 tiles 287 us, 384 of 192 columns 254; 256
// rows, FC1: 96 tiles split in two 114 us, 192 of 128 columns 101).  Once x is beyond
// the L2s, what narrower tiles read more of it is priced at 20 TB/s (4,096 rows,
// FC2: 1,086 us with 256 columns, 1,108 with 192).
inline GemmPlan tile_plan(int64_t M, int64_t N, int64_t K, const KSplits& ks, int64_t cus, double limit) {
  const bool half = M <= kGemmHalfM;
  GemmPlan best{};
  bool found = false;
  double bytes0 = 0.0;
  for (int i = half ? 0 : 1; i < (half ? 1 : 4); ++i) {
    const TileShape& t = kTileShapes[i];
    GemmPlan p{GemmRoute::kTiles, i, ceil_div(M, t.bm), ceil_div(N, t.bn), 1, 0, 0, 0.0};
    // rows past M multiply zeros, which takes less power (136 rows, FC1 of the
    // 6144-wide layer: 1.28 us a step against 1.5 at 256 rows; no difference at 128 columns)
    const double load = i == 1 || i == 2 ? 0.7 + 0.3 * (double)M / (double)(p.mtiles * t.bm) : 1.0;
    p.splits = tile_splits(p.mtiles * p.ntiles, ks, M, N, cus, t, load, limit, &p.us);
    if (p.us < 0.0) continue;
    const double bytes = (double)K * ((double)p.ntiles * (double)M * 2.0 + (double)p.mtiles * (double)N);
    if (i <= 1) bytes0 = bytes;
    else if (M * K * 2 > 16 << 20) p.us += (bytes - bytes0) / 20e6;
    if (!found || p.us < best.us) best = p;
    found = true;
  }
  best.grid = best.mtiles * best.ntiles * best.splits;
  return best;
}

// Whether and how k_dqrows runs M rows (kind < 0: not).  Each workgroup reads its rows
// of x once over all of K, so the weight rows per workgroup (16 NG) are as many as
// leave about one workgroup per CU (N / 256, up to 96): 16 rows, QKV of the
// 6144-wide layer 32.7 us with 384 workgroups of 48 weight rows, 28.3 with 231 of 80;
// 64 rows 49.5 and 41.  Past 32 rows the candidates' times are modelled as a launch
// and the busiest CU's bytes of codes and x at the rate that the variant reaches:
//   4 us + ceil(workgroups / CUs) (16 NG + 32 MT) K / rate
// rate 45 bytes per ns where several workgroups or 8 waves share a CU, 31-34 for
// the wide ones (measured: 64 rows, QKV of the 6144-wide layer 41 us, modelled 42;
// FC1 49, 48; attention output 23, 26; FC1 of the 2048-wide layer 11.5, 11.3).
// The tiled kernels' model (tile_plan) gives 49, 62, 30 and 22 there, 50, 63, 28
// and 20 measured.
inline GemmPlan rows_plan(int64_t M, int64_t N, int64_t K, int lgB, int64_t cus, double limit) {
  GemmPlan best{};
  best.route = GemmRoute::kRows;
  best.kind = -1;
  // (start: us before the first step)
  auto take = [&](int mt, int ng, int w, bool xl, int few, double rate, double start = 4.0) {
    if (((16 * ng * K) >> lgB) + 1 > kScaleLds) return;  // its rows' scales have to fit LDS
    const int64_t ngroups = ceil_div(N, 16 * ng), mgroups = ceil_div(M, 16 * mt), wgs = ngroups * mgroups;
    if (few >= 0 && (wgs <= cus) != (few == 1)) return;
    // the first variant of these tiles whose sums are short enough, of two sets only
    // where one workgroup a CU is all there are
    int kind = -1;
    for (int i = 0; i < kRowsKinds && kind < 0; ++i) {
      const RowsVariant& v = kRowsVariants[i];
      if (v.mt == mt && v.ng == ng && v.w == w && v.xl == xl && !v.ks &&
          sum_drift((double)K / (w * v.sets), 0.0, w) <= limit &&
          !(mt == 4 && (ng == 3 || ng == 4) && v.sets == 2 && wgs > cus))
        kind = i;
    }
    if (kind < 0) return;
    const int64_t xbytes = xl ? 2 * M : 32 * mt;  // of a column of x
    double us = (double)(ceil_div(wgs, cus) * (16 * ng + xbytes) * K) / rate * 1e-3;
    // the codes at HBM's rate, of which a part of the GPU has its part
    const double hbm = (double)N * (double)K / 5.5e6 * 256.0 / (double)cus;
    if (M <= 16 && us < hbm) us = hbm;
    us += start;
    if (best.kind < 0 || us < best.us)
      best = {GemmRoute::kRows, kind, mgroups, ngroups, 1, ceil_div(ngroups, kRowsXcds) * kRowsXcds * mgroups, 0, us};
  };
  if (K == 0) return best;
  const int64_t per_cu = ceil_div(N, 16 * cus);  // weight-row tiles a CU where each has one workgroup
  if (M <= 16 && M * K * 2 <= kXLds) {
    // 48 weight rows where N leaves two workgroups a CU or nearly so, else 16
    // (1 row: N = 24576 27.5 us, 29.0 with 32 weight rows; N = 6144 11.7, 13.0
    // with 32; N = 2048, K = 2048 5.1, 6.7)
    if (N >= 64 * cus) take(1, 3, 8, true, -1, 45.0);
    else take(1, 1, 8, true, -1, 45.0);
  } else if (M <= 32) {
    // (2 weight-row tiles at 16 waves where N is small: N = 6144 13.9 us, 16.5 with one)
    const int mt = M <= 16 ? 1 : 2;
    if (per_cu > 2) take(mt, (int)(per_cu < 6 ? per_cu : 6), 8, false, -1, 34.0);
    if (best.kind < 0 && mt == 1) take(1, 2, 16, false, -1, 37.0, 2.4);
    if (best.kind < 0 && mt == 2) take(2, 2, 8, false, -1, 45.0);
  } else {
    // 8 waves where each CU has one workgroup at most, else 4 (128 rows,
    // N = 8192, K = 2048: 16.4 us, 19.3 with 8; 64 rows, N = K = 6144: 23.9 and 22.8)
    take(4, 2, 8, false, 1, 45.0);
    take(4, 2, 4, false, 0, 45.0);
    take(4, 3, 4, false, -1, 45.0);
    take(4, 4, 4, false, -1, 34.0);
    take(4, 5, 4, false, -1, 34.0);
    take(4, 6, 4, false, -1, 31.0);
  }
  if (M > 32) return best;
  if (M <= kGemvRows && K >= 4 * N) best.kind = -1;  // too few workgroups take K whole
  // K long against N leaves few workgroups that take it whole: 96 weight rows and
  // as many ranges of K as fill the CUs (of 1024 at least), added into a zeroed y (6144
  // x 24576: 64 groups of rows, 4 ranges; 16 rows 48.1 us on the weight-streaming kernel
  // that splits K 24 ways, 39.0; 32 rows 51.8 on the tiled one, 40.9).  Past 32 rows
  // the tiled kernel is even.
  const int mt = M <= 16 ? 1 : 2;
  const int64_t ngroups = ceil_div(N, 96);
  int64_t ks = cus / (ceil_div(ngroups, kRowsXcds) * kRowsXcds);  // (a group's ranges run on one XCD)
  if (ks > K / 1024) ks = K / 1024;
  if (ks < 2) return best;
  const double us = 5.9 + (double)mt + (double)((96 + 16 * mt) * K) / (double)ks / 22.1e3 +
                    (double)M * (double)N * (double)ks * kGemmAtomicUs;
  int kind = kRowsKinds - 1;
  while (kRowsVariants[kind].mt != mt) --kind;
  if (((K / ks + 128) >> lgB) + 2 <= kRangeScales && 96 * K < (int64_t(1) << 30) &&
      sum_drift((double)K / (double)(ks * 8 * kRowsVariants[kind].sets), (double)ks, 8.0) <= limit &&
      (best.kind < 0 || us < best.us))
    best = {GemmRoute::kRows, kind, 1, ngroups, ks, ceil_div(ngroups, kRowsXcds) * kRowsXcds * ks, 0, us};
  return best;
}

// The kernel that runs M rows against an N x K weight in blocks of 2^lgB.  Few rows:
// k_dqrows where it has a plan (past 16 rows: where that plan's modelled time is the
// lower).
inline GemmPlan gemm_plan(int64_t M, int64_t N, int64_t K, int lgB, int64_t cus) {
  if (M <= kGemvRows) {
    // the weight-streaming kernel: its launches, its codes and its additions (16 rows
    // of K = 4096 against N = 2048: 8.6 us, 9.5 on k_dqrows; N = 4096: 12.9 and 9.9)
    GemmPlan gemv{GemmRoute::kGemv, 0, 1, ceil_div(N, 64), 1, 0, gemv_range(N, K), 0.0};
    gemv.splits = K > gemv.kc ? ceil_div(K, gemv.kc) : 1;
    gemv.grid = gemv.ntiles * gemv.splits;
    gemv.us = 5.6 + ((double)N * (double)K / 4.8e6 + (double)M * (double)N * (double)gemv.splits * 3e-6) *
                        256.0 / (double)cus;
    const double limit =
        kDriftSlack * sum_drift((double)(gemv.kc < K ? gemv.kc : K), (double)gemv.splits, 0.0);
    const GemmPlan rows = rows_plan(M, N, K, lgB, cus, limit);
    return rows.kind >= 0 && rows.us < gemv.us ? rows : gemv;
  }
  if (K > kGemmPpMaxK) {
    // one plain kernel, 64-bit addresses
    const int64_t mt = ceil_div(M, 256), nt = ceil_div(N, 256);
    return {GemmRoute::kPlain, 0, mt, nt, 1, mt * nt, 0, 0.0};
  }
  const KSplits ks = k_splits(K);
  const double limit = drift_limit(M, N, ks, cus);
  const GemmPlan rows = rows_plan(M, N, K, lgB, cus, limit), tiles = tile_plan(M, N, K, ks, cus, limit);
  return rows.kind >= 0 && rows.us < tiles.us ? rows : tiles;
}

}  // namespace zq
