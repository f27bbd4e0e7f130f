// Tile shape of a bf16 product on the large-tile kernel (host arithmetic only).
#pragma once

#include <algorithm>
#include <cmath>

namespace lx {

struct TilePick {
  int bm, bn;
  double us;       // predicted time
  double base_us;  // the same of 256 x bn0
  bool base;       // 256 x bn0 was kept
};

// The rows of N nodes (T tokens, k experts each) against weights of `work` of
// them, ncol columns, depth K: bm x bn. bn0 is the column count of the 256-row
// tiles that suit the product on a full chip (256, or less where its columns
// fill no 256); part_cols: tiles must not straddle the two parts of that many
// columns (0: they may).
//
// 256 x bn0 does the most MFMA work per byte staged and is kept where it gives
// every compute unit an item (T = 4096 and 8192, f = 576 to 1600: the other shapes
// took 0.8 to 3 times its time on the wide products, by how their last round
// fills; 256 columns for the 64 to 128 of a low-rank input took 1.6 times, 118
// against 74 us). With fewer items a launch lasts
// as long as one item, so smaller tiles win as long as they still fit in few
// rounds of 256 items. A round takes `item` + `slab` us per 64-wide slab, of the
// rows or of padding alike (launches of 100 to 2000 items of 1 to 50 slabs came
// within 15% of that). The tiles per node follow from uniform routing: T (1 - (1
// - 1/N)^k) rows and their binomial deviation, or 10% of the rows more than that
// for a router that is not uniform; a smaller shape has to win by a tenth under
// whichever of the two is worse for it.
// Measured, 256 x bn0 against the chosen shape, us (d = 2048, 16 anchors of 128
// experts, k = 8): f = 768, T = 237 gate|up 54 -> 32, down 44 -> 27; T = 400 55 ->
// 35, 45 -> 31; f = 1280, r = 32, T = 400 down 69 -> 47, low-rank input 33 -> 23. At
// T = 700 gate|up needs 12 x 48 items of 128 x 128 (three rounds): 57 against 78,
// and 256 x 256 is kept.
inline TilePick pick_tile(int N, int work, int T, int k, int ncol, int K, int part_cols, int bn0) {
  static constexpr struct {
    int bm, bn;
    double slab, item;
  } kShapes[] = {{256, 256, 1.60, 5.0}, {256, 128, 0.98, 3.4}, {256, 64, 0.92, 3.0},
                 {128, 128, 0.85, 3.0}, {128, 64, 0.58, 2.2}};
  const double mean = T * (1.0 - std::pow(1.0 - 1.0 / N, k));
  // expected tiles of a node: sum over i of P(rows > i bm)
  auto tiles = [&](int bm, double sd) {
    if (sd >= bm) return mean / bm + 0.5;
    int i = std::max(1, (int)((mean - 4.0 * sd) / bm));
    double t = i;
    for (; i * bm < mean + 4.0 * sd; ++i) t += 0.5 * std::erfc((i * bm + 0.5 - mean) / (sd * std::sqrt(2.0)));
    return t;
  };
  auto items = [&](int bm, int bn, double sd) { return work * tiles(bm, sd) * ((ncol + bn - 1) / bn); };
  const double sd1 = std::sqrt(std::max(0.0, mean * (1.0 - mean / T))) + 1e-9;
  const double sd2 = sd1 + 0.1 * std::min(mean, T - mean);
  TilePick p{256, bn0, 0.0, 0.0, true};
  const double base_items = items(256, bn0, sd1);
  const bool full = base_items >= 256.0;
  for (const auto& c : kShapes) {
    const bool base = c.bm == 256 && c.bn == bn0;  // (listed before the others of at most its columns)
    if (c.bn > bn0 || (part_cols && part_cols % c.bn) || (full && !base)) continue;
    auto us = [&](double n) { return std::max(1.0, std::ceil(n / 256.0 - 0.05)) * (K / 64 * c.slab + c.item); };
    const double u1 = us(items(c.bm, c.bn, sd1)), u2 = us(items(c.bm, c.bn, sd2));
    if (base) {
      p.us = p.base_us = std::min(u1, u2);
    } else if (std::max(u1, u2) < 0.9 * p.base_us && std::max(u1, u2) < p.us) {
      p.bm = c.bm;
      p.bn = c.bn;
      p.us = std::max(u1, u2);
      p.base = false;
    }
  }
  return p;
}

}  // namespace lx
