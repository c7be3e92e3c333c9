// Levels of a top-k sweep: which labels each level takes.  Host arithmetic only, no HIP.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>

namespace elmo {

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
    return std::min<int64_t>(L, (int64_t)((double)level0 * std::pow(growth, level) + 255.0) / 256 * 256);
  }
};
inline TopkLevels topk_levels(int64_t L, int Bp, int k) {
  TopkLevels t{L, std::min<int64_t>(L, kTopkLevel0), 0, 1.0};
  const double ratio = (double)L / (double)t.level0;
  double most = topk_most_growth(Bp, k);
  // A level saved is a launch that does not fill the chip and a select, 35-45 us at 256 rows.  131072 BF16 labels, B = 256,
  // k = 100: 175 us at most 4-fold, 150 us at 5.7; 20000 labels, B = 1024: 111 and 94 us.  Where the product is
  // everything, the appends (device-scope additions) weigh more: 3 M labels, B = 1024: 2.18 and 2.22 ms.
  if (Bp > 128) most = std::min(most, L * Bp >= (int64_t)1 << 31 ? 4.0 : 5.7);
  t.n = (int)std::ceil(std::log(ratio) / std::log(most) - 1e-9);
  if (t.n > 0) t.growth = std::pow(ratio, 1.0 / t.n);
  return t;
}

}  // namespace elmo
