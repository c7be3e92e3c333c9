// Levels of a top-k sweep, which labels each level takes, and the scratch of a call.  Host arithmetic only, no HIP.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>

namespace elmo {

constexpr int kTopkMaxK = 128;                     // entries selected per sweep (one page)
constexpr int kTopkCntStride = 32;                 // ints between two rows' candidate counters: one 128-byte line each, so that the
                                                   // atomic additions of different rows do not queue up on the same few lines
constexpr int kTopkRows = 64;                       // query rows per workgroup
constexpr int kTopkCand = 4096;                    // candidate list length per row of a batch padded to whole 256-row tiles
constexpr int kTopkLevel0 = 4096;                  // labels of the first level
static_assert(kTopkLevel0 <= kTopkCand, "the first level writes one slot per label");
// A batch of at most 128 rows (padded) has the lists of the 128 rows that the padding to 256 adds as well.
inline int topk_list(int Bp) { return Bp <= 128 ? 2 * kTopkCand : kTopkCand; }

// Labels seen after a level / labels seen before it, at most.  A level appends about k (growth - 1) scores per row if
// the scores stand in no order along the label axis -- but labels are often numbered by frequency, and weight norms
// follow it.  So a level is kept so short that its scores may be twice as spread as the 4096 before it and still fit the
// lists, for the lowest of a batch of thresholds (one row in a thousand): with z the standard normal deviate that
// 4096 scores exceed k times on average, (growth - 1) 4096 P(N(0, 2) > z) stays below the list.  The power below
// is that bound for k = 1 .. 128, within 16 % on the safe side.  A row whose list overflows is recomputed over all
// labels by the slow path.  670091 BF16 labels, k = 10, one query, scores twice as spread after label 4096: 1432 us with
// one level of 12.8-fold growth after the first and 4096 slots, 468 us with levels of 4-fold growth, 224 us here (216 us
// with even scores); k = 34, 128 queries: 4830, 531 and 481 us.
inline double topk_most_growth(int Bp, int k) { return 1.0 + 13.0 * (topk_list(Bp) / kTopkCand) * std::pow((double)k, -0.2); }

// The levels after the first: `n` of them, each `growth` times the labels seen before.
struct TopkLevels {
  int64_t L, level0;
  int n;
  double growth;
  // labels seen when `level` (0: the first) has been taken
  int64_t end(int level) const {
    if (level == n) return L;
    if (level == 0) return level0;
    return std::min<int64_t>(L, (int64_t)((double)level0 * std::pow(growth, level) + 255.0) / 256 * 256);
  }
};
// As few levels as the lists allow for a batch of at most 128 rows, which pays for launches (one query or 128, 20000 .. 1.5 M BF16
// labels: a level more is 5 .. 24 us).  A larger batch also pays for appends, device-scope additions, and a level of it
// may end just above a whole wave of 256 x 256 tiles.  So every number of levels is priced, in us: launch and select of a
// level, its waves of tiles of `slabs` K slabs (as the step's logits), and its appends, which a wave hands over together the
// more of them there are.  575 shapes (160 .. 2048 rows, 20000 .. 3 M labels, k = 1 .. 100, both types, d = 768): 0.15 % above
// the best number of levels on average, 6 % at most; with a fixed limit of 5.7 2.6 % and 38 %.  BF16, 140000 labels (two
// levels / three): 256 rows, k = 10 113 / 138 us; 1024 rows, k = 34 328 / 293; 131072 labels, 1024 rows, k = 100 381 / 356.
inline TopkLevels topk_levels(int64_t L, int Bp, int k, int slabs) {
  TopkLevels t{L, std::min<int64_t>(L, kTopkLevel0), 0, 1.0};
  const double ratio = (double)L / (double)t.level0;
  const int least = (int)std::ceil(std::log(ratio) / std::log(topk_most_growth(Bp, k)) - 1e-9);
  if (least <= 0) return t;
  const int64_t tiles_b = (Bp + 255) / 256;
  double cheapest = 0.0;
  for (int n = least; n <= (Bp <= 128 ? least : least + 6); ++n) {
    TopkLevels c{L, t.level0, n, std::pow(ratio, 1.0 / n)};
    if (n > least && c.growth < 2.25) break;                   // (beyond what was measured)
    double price = n * (16.0 + 0.001 * Bp * std::sqrt((double)k) * (c.growth - 1.0));
    for (int lv = 1; lv <= n; ++lv) price += (double)((((c.end(lv) - c.end(lv - 1) + 255) / 256) * tiles_b + 255) / 256) * (6.0 + 1.4 * slabs);
    if (n == least || price < cheapest) { cheapest = price; t = c; }
  }
  return t;
}

// Label segments per 64-row group: enough workgroups to fill the chip, at most 64 lists to merge.
inline int topk_segments(int tiles_b) { return std::max(1, std::min(64, 512 / tiles_b)); }

// Main-path scratch: thresholds, counters, overflow flags and candidate lists per (padded) row.
inline size_t topk_main_rows(int Bp_max) { return (size_t)(Bp_max + 255) / 256 * 256; }
static_assert(256 * kTopkCand >= 128 * 2 * kTopkCand, "the longer lists of at most 128 rows fit where those of 256 do");
inline size_t topk_main_bytes(int Bp_max) { return topk_main_rows(Bp_max) * (24 + (size_t)kTopkCntStride * 4 + (size_t)kTopkCand * 8) + 1024; }

// Bytes of per-segment partial lists for any batch of at most Bp_max rows, plus the main path's.
inline size_t topk_scratch_bytes(int Bp_max, int64_t /*chunk*/) {
  const int tb_max = (Bp_max + kTopkRows - 1) / kTopkRows;
  size_t lists = 0;
  for (int tb = 1; tb <= tb_max; ++tb) lists = std::max(lists, (size_t)tb * kTopkRows * topk_segments(tb));
  return lists * kTopkMaxK * 8 + topk_main_bytes(Bp_max);
}

}  // namespace elmo
