// Host side of a head: its workspace and the passes of a step.  Arithmetic only, no HIP.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <utility>

#include "../../include/elmo_head.h"
#include "topk_levels.h"

namespace elmo {

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline int round_up(int x, int m) { return (x + m - 1) / m * m; }

// Workspace plan: byte offsets of every region (Section 4.2/4.4: only one chunk's logit-gradient
// buffer is ever alive; everything else is O(max_B * d) or O(L / 128) integers).
struct Plan {
  int64_t L; int d; int fmt; int64_t chunk; int maxB; int64_t max_nnz; uint32_t flags;
  int64_t kahan_rows;                   // leading label rows that carry compensation (0 without ELMO_KAHAN)
  float weight_decay;                   // L2 term of the update, 0 = none
  uint32_t drop_thresh;                 // classifier dropout: weights dropped with probability drop_thresh / 256, 0 = none
  int Bp_max, tiles_b_max, ntiles;      // padded batch, batch tiles, 128-label tiles of the whole head
  int dx_rows;                          // rows of FP32 input-gradient partials (slices x padded batch)
  size_t off_xq, off_xt, off_g, off_dx, off_loss, off_cnt, off_ptr, off_cur, off_pos, off_flag, off_topk, total;
  size_t W_bytes, comp_bytes;
};

// Sizes and offsets from the first two lines of a plan.
inline void lay_out(Plan& p) {
  p.Bp_max = round_up(p.maxB, 64);
  p.tiles_b_max = (p.Bp_max + 255) / 256;      // 256-sample tiles of the matrix products
  p.ntiles = (int)((p.L + 127) / 128);
  const int tiles_j = (p.d + 255) / 256;           // 256-column tiles of the input-gradient product
  // slices x padded batch of the input-gradient partials: about one workgroup per CU
  p.dx_rows = std::min(65536 / tiles_j + 256 * p.tiles_b_max + 256, 64 * 256 * p.tiles_b_max);
  if (p.d % 256 == 0) p.dx_rows = std::max(p.dx_rows, std::max(1, 256 / (p.d / 256)) * 128);   // small-batch path: one 128-row slice per label group
  const int64_t chunk_eff = std::min<int64_t>(p.chunk, (p.L + 127) / 128 * 128);
  size_t o = 0;
  p.off_xq = o;  o += align256(p.fmt == ELMO_FP8_E4M3 ? (size_t)p.Bp_max * p.d : 0);
  p.off_xt = o;  o += align256((size_t)p.d * p.Bp_max * 2);
  p.off_g = o;   o += align256((size_t)chunk_eff * p.Bp_max * 2);   // whole blocks of 32 labels, read and written as such
  p.off_dx = o;  o += align256((size_t)p.dx_rows * p.d * 4);
  p.off_loss = o; o += align256((size_t)p.ntiles * p.tiles_b_max * 4);
  p.off_cnt = o; o += align256((size_t)(p.ntiles + 1) * 4);
  p.off_ptr = o; o += align256((size_t)(p.ntiles + 1) * 4);
  p.off_cur = o; o += align256((size_t)(p.ntiles + 1) * 4);
  p.off_pos = o; o += align256((size_t)p.max_nnz * 8);
  p.off_flag = o; o += 256;
  p.off_topk = o; o += align256(topk_scratch_bytes(p.Bp_max, chunk_eff));
  p.total = o;
  p.W_bytes = (size_t)p.L * p.d * (p.fmt == ELMO_FP8_E4M3 ? 1 : 2);
  p.comp_bytes = (size_t)p.kahan_rows * p.d * 2;
}

// Labels per pass of the step and where its logit gradients live.  The chunk bounds the memory that the
// gradients take, not the work of a launch: a pass may take more labels where the workspace holds
// their gradients anyway -- the chunk's own region when the batch is smaller than max_B, or the top-k
// scratch, which is idle during a step.  Short launches cost most: L = 8192, B = 64 in chunks of 2048 spent
// 54 of 61 us in eight kernels of 6-7 us each that leave most of the chip idle, one pass takes 26 us.
// So every number of passes that the room allows is priced by what the backward kernels of the step (below) have to do and the cheapest is
// taken, the chunk itself included.
//   kSeparate has whole waves of 256 x 256 tiles to think of (one workgroup per CU): 677016 labels at
//     B = 2733 in passes of 16384 (192 update tiles) take 10.06 ms and in passes of 22656 (267, a second
//     wave of 11) 10.85 ms.  Its prices are the waves of the launches (microseconds per tile and K slab as measured at d = 768: a tile's epilogue
//     and its slabs, and what the launches cost before and after their tiles, 15 us, 13 without the input gradient where dX is not asked
//     for: 60000 E4M3 labels at B = 3000 506 us in the passes that are cheapest with it, 480 without).
//   kOnePass128 is a pass over the weights whatever the split; a pass costs its launches and the planes of partial sums that it reads and
//     writes (20 us), the waves of its logits tiles (half a tile each, the rest hides behind other work; up to 128 tiles of 256 labels take the small
//     ones, two to a CU), and the label tiles of its longest group.  1031 heads, 129 to 256 rows and 384 or 640 columns at fewer, each at up to 12 splits:
//     the split with this price is 0.4 % slower than the best on average (worst 13 %), priced as kSeparate 1.5 % (15 %), the fewest passes
//     1.3 % (19 %).  1202307 E4M3 labels, d = 768, B = 129: 28 passes 2567 us, 23 passes 2323.  (What it cannot see: for some numbers of label tiles to a
//     group the groups' strides meet in memory, 58 or 59 tiles of 640 columns with compensation 15 % slower than 57 or 60.)
//   kOnePass256 (at most 128 rows) takes the fewest passes, of equal size.
// Offered are passes of equal size, and for kSeparate passes of whole waves of update tiles (L = 131072, B = 256: 171 + 171 + 170 label tiles
// 442 us, 170 + 170 + 172 420 us), for kOnePass128 of whole waves of small logits tiles, the last of which takes what is
// left if that fits.  No pass but the last is smaller than the chunk.  The prices only rank the splits of one head.  Results do
// not depend on the split: every label's quantities depend on its own weight row only, and dX is summed in FP32.
// Passes of at most this many 256 x 256 logits tiles take 128 x 128 tiles at batches above 128 too: half of the CUs
// would have no tile, and four times the tiles, two on a CU at once, are one wave up to here.  32768 BF16 labels,
// B = 256, d = 768: 30.4 -> 24.8 us; 60000 E4M3 labels, d = 512, B = 160, whole step: 134 -> 120 us; with a second wave
// of the small tiles the large ones win (43776 labels: 34 us against 43 us).
constexpr int kLogitsSmallGrid = 128;
enum Backward { kSeparate, kOnePass256, kOnePass128 };
struct Pass {
  int64_t labels, most;      // labels of a pass; what is left at the end is one pass if it is no more than `most`
  size_t off_g, slots;
  int64_t take(int64_t left) const { return left <= most ? left : labels; }
  int64_t largest(int64_t L) const {
    const int64_t before = L > most ? (L - most + labels - 1) / labels : 0;
    return std::max(before ? labels : 0, L - before * labels);
  }
};
inline int label_groups_128(const Plan& p) { return std::max(1, std::min(256 / (p.d / 128), p.dx_rows / 256)); }
inline Pass choose_pass(const Plan& p, int Bp, Backward kernels, bool want_dx) {
  // tile losses of 128 x 128 logits tiles at a batch above 128 go to the end of the top-k scratch (0: no room)
  const size_t slots = align256((size_t)p.ntiles * ((Bp + 127) / 128) * 4);
  Pass best{p.chunk, p.chunk, p.off_g, p.total - p.off_topk >= slots ? p.total - slots : 0};
  if (p.chunk >= p.L) return best;
  const int esz = p.fmt == ELMO_FP8_E4M3 ? 1 : 2;
  const int64_t tiles_b = (Bp + 255) / 256, tiles_j = (p.d + 255) / 256, slices = std::max<int64_t>(1, 256 / (tiles_b * tiles_j));
  const int groups = label_groups_128(p);
  auto launches = [&](int64_t n, bool small_logits) {
    const int64_t lt = (n + 255) / 256;
    if (kernels == kOnePass128) {
      const int64_t tiles = (n + 31) / 32;
      const double waves = Bp <= 128 ? (double)(((n + 127) / 128 + 511) / 512) : small_logits ? 0.8 : (double)((lt + 255) / 256);
      return 20.0 + waves * (3.0 + 0.7 * (p.d * esz / 128)) + (double)((tiles + groups - 1) / groups);
    }
    return (double)((lt * tiles_j + 255) / 256) * (10.0 + 1.4 * (Bp / 64)) + (double)((lt * tiles_b + 255) / 256) * (6.0 + 1.4 * (p.d * esz / 128)) +
           (want_dx ? 1.4 * (double)((lt * 4 + slices - 1) / slices) + 15.0 : 13.0);
  };
  auto price = [&](int64_t n, int64_t most) {
    const int64_t before = p.L <= most ? 0 : (p.L - most + n - 1) / n, last = p.L - before * n;
    const bool small_logits = best.slots && (std::max(before ? n : 0, last) + 255) / 256 * tiles_b <= kLogitsSmallGrid;
    return (double)before * launches(n, small_logits) + launches(last, small_logits);
  };
  double cheapest = kernels == kOnePass256 ? 0.0 : price(p.chunk, p.chunk);
  for (auto [off, end] : {std::pair<size_t, size_t>{p.off_g, p.off_dx}, {p.off_topk, best.slots}}) {
    if (end < off) continue;
    const int64_t room = (int64_t)((end - off) / ((size_t)Bp * 2)) / 128 * 128;
    if (room <= p.chunk) continue;
    const int64_t least = (p.L + room - 1) / room;
    auto consider = [&](int64_t labels) {
      if (labels <= p.chunk || labels > room) return;
      const double t = price(labels, room);
      if (t > cheapest + 1e-6 || (t > cheapest - 1e-6 && (kernels == kSeparate || labels <= best.labels))) return;
      cheapest = t;
      best = {labels, room, off, best.slots};
    };
    if (kernels == kOnePass256) {              // no tiles to fill: the fewer launches the better
      const int64_t labels = ((p.L + least - 1) / least + 127) / 128 * 128;
      if (labels > best.labels) best = {labels, labels, off, best.slots};
      continue;
    }
    for (int64_t passes = least; passes < least + 64; ++passes) consider(((p.L + passes - 1) / passes + 127) / 128 * 128);
    for (int64_t waves = 1; waves <= 64; ++waves) consider(kernels == kSeparate ? 256 * waves / tiles_j * 256 : 32768 * waves);
  }
  return best;
}

// What a step launches for a batch padded to Bp rows: its passes, the kernels of their backward half and how those split the labels.
//   kOnePass256: input gradient and update in one pass over the weights, tiles of 32 labels x 256 columns (k_dx_update), at most 128 rows.
//     With dropout that kernel keeps a masked copy of the W tile in LDS, which does not fit next to BF16 weights with
//     compensation: without an input gradient that one mode takes the separate kernels.
//   kOnePass128: the same in tiles of 128 columns (k_dx_update_wide), at most 256 rows, as far as the planes of partial sums have room for groups that
//     fill the chip (d = 384: 64 groups of 3 workgroups; d = 128, 64 workgroups, takes the separate kernels), and where an input
//     gradient is asked for: the update alone has no second read of W to save (21293 E4M3 labels, B = 134: 39 us, 45 us there).
//     At most 128 rows take it where 256 does not divide d (300000 E4M3 labels, d = 640, B = 128: separate kernels 409 us, 283 us there) and where
//     a workgroup has no more than four of its tiles (16384 E4M3 labels, d = 256, B = 64: 256 columns 29.5, 128 columns 25.7 us;
//     16384 x 768, twelve tiles: 35.7 and 36.1; 1 M labels, B = 128, with compensation: 1406 and 1472).
//   kSeparate: input-gradient product, then update (k_dx, k_update).
struct StepPlan {
  Pass ps;
  Backward kernels;
  int slices;                     // kSeparate: label slices of the input-gradient product
  int col_blocks, label_groups;   // one pass: workgroups side by side over the columns, and the most over the labels
  int planes, plane_rows;         // of partial sums of dX: what the step's first launch writes and the end adds up
  bool one_pass() const { return kernels != kSeparate; }
  int64_t tiles_per_group(int64_t tiles) const { return (tiles + label_groups - 1) / label_groups; }
  int groups(int64_t labels) const {
    const int64_t t = (labels + 31) / 32, per = tiles_per_group(t);
    return labels > 0 ? (int)((t + per - 1) / per) : 0;
  }
};
inline StepPlan plan_step(const Plan& p, int Bp, bool want_dx) {
  StepPlan s;
  const int d = p.d, Bp256 = round_up(Bp, 256), tiles_b = Bp256 / 256, tiles_j = (d + 255) / 256;
  const bool no_room = p.drop_thresh && p.fmt != ELMO_FP8_E4M3 && (p.flags & ELMO_KAHAN);
  const bool narrow = Bp <= 128 && d % 256 == 0 && !no_room;
  const int wide_groups = label_groups_128(p);
  const bool may_wide = want_dx && Bp <= 256 && wide_groups * (d / 128) >= 192;
  s.ps = choose_pass(p, Bp, narrow ? kOnePass256 : may_wide ? kOnePass128 : kSeparate, want_dx);
  const int64_t most = std::min<int64_t>(s.ps.labels, p.L), wide_tiles = (most + 31) / 32 * (d / 128);
  const bool wide = may_wide && (!narrow || wide_tiles <= 4 * 256);
  s.kernels = wide ? kOnePass128 : narrow ? kOnePass256 : kSeparate;
  s.col_blocks = wide ? d / 128 : d / 256;
  s.label_groups = wide ? wide_groups : narrow ? std::max(1, 256 / s.col_blocks) : 0;    // widths above 65536: one group
  // slices: at most one 512-thread workgroup per CU, so the
  // whole grid is resident at once (256 CUs) and no second, nearly empty round of workgroups runs
  s.slices = std::min(std::max(1, 256 / (tiles_b * tiles_j)), p.dx_rows / Bp256);
  s.slices = std::max(1, std::min({s.slices, 64, (int)((most + 63) / 64)}));
  // a one-pass kernel uses as many planes as its largest launch has label groups
  s.planes = s.one_pass() ? 1 : s.slices;
  if (s.one_pass())
    for (int64_t c0 = 0; c0 < p.L; c0 += s.ps.take(p.L - c0)) {
      const int64_t n = s.ps.take(p.L - c0), head = std::max<int64_t>(0, std::min(n, p.kahan_rows - c0));
      s.planes = std::max({s.planes, s.groups(head), s.groups(n - head)});
    }
  s.plane_rows = s.kernels == kOnePass256 ? 128 : Bp256;
  return s;
}

}  // namespace elmo
