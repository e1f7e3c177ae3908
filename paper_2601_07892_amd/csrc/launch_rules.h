// Rules by which the host picks a launch's shape from its sizes, and by which
// workgroups find their part of it: plain C++ (no HIP), so that they can be
// checked on the CPU.
#pragma once

#include <cstdint>

namespace sherry {

constexpr int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Activation quantization: inputs of kStreamBytes and more are read past the
// caches (non-temporal).  Usually the operation before has just written the
// input.  Time with streaming against without, after a kernel that wrote x from
// one tensor, from two, and in place, and with x evicted (rows of 2048 .. 14336
// values): 12 MB +1%, +5%, +6%, -17%; 20 MB +2%, 0%, +14%, +2%; 32 MB -1%, -7%, +14%,
// -11%; 64 MB -5%, -8%, -3%, -4% (13.9 -> 12.9 us at 1953 x 8192); 96 MB -6%,
// -20%, -8%, -20%; 160 MB -23%, -26%, -10%, -8% (33.7 -> 25.4 us at 4882 x 8192).
constexpr int64_t kStreamBytes = int64_t(64) << 20;
constexpr bool quant_streams(int64_t rows, int64_t k) { return 4 * rows * k >= kStreamBytes; }

// Threads per row and float4 pieces per thread (0: two passes over the row) of
// the quantization of `rows` rows of up to k values.  512 threads past 8192
// values (1000 x 30000 51.7 -> 25 us, 64 x 14336 6.1 -> 4.7), except where the
// launch, one row per workgroup, would not fit the 2^32 - 1 threads of a grid.
struct QuantShape {
  int threads, pieces;
};
constexpr QuantShape quant_shape(int64_t rows, int64_t k) {
  if (k <= 8192) return {256, k <= 2048 ? 2 : k <= 4096 ? 4 : 8};
  if (rows * 512 > int64_t(UINT32_MAX)) return {256, k <= 16384 ? 16 : 0};
  return {512, k <= 16384 ? 8 : k <= 32768 ? 16 : 0};
}

// ---- 5-16-token window kernel: K in four parts ------------------------------

// Grouped launches of up to kSmFoldBlocks prepared blocks (of four tiles) run
// four workgroups per block, each of one tile with a quarter of its K per wave,
// for the products whose rows gain by it (sm_splits); the blocks of the others are
// run by one of the four, one tile per wave.  Time over whole rows at 12 tokens,
// rows of 1 / 4 / 8 / 16 / 32 / 64 units: up to 64 blocks 1.06 / 0.89 / 0.75 / 0.58 /
// 0.48 / 0.41 (18.2 -> 7.5 us), left whole 1.00; 128 blocks 1.17 / 1.01 / 0.85 / 0.69
// / 0.61 / 0.56 (two workgroups per CU, one round); 192 blocks 1.74 / 1.43 / 1.22 /
// 0.99 / 0.91 / 0.87, left whole 1.15 .. 1.28; 256 blocks 1.80 / 1.57 / 1.38 / 1.16 /
// 1.07 / 1.00.  (Launches that mix long rows with short ones gain more: 158 blocks
// 47 -> 19 us.)  Per-group scales: parts of whole chunks of four units.
constexpr int64_t kSmFoldBlocks = 192;
constexpr bool sm_splits(int64_t units, int64_t blocks, bool group_scales) {
  return units >= (blocks > 128 ? 8 : 4) + (group_scales ? 4 : 0);
}
// The workgroup of a block's four that runs it whole.  Workgroups go to the 8 XCDs
// in turn and there to the four shader engines in turn, so the choice varies with
// both (always the first: 184 blocks 20 -> 44 us).
constexpr int sm_whole_sub(int block) {
  const int j = block >> 1;
  return (j ^ (j >> 2) ^ (j >> 4)) & 3;
}

// ---- register-decoded products: shapes of a workgroup -----------------------

// Tokens x 64-row tiles of a workgroup, and the parts its tiles' K is split in.
enum WideShape : int {
  kWideLong, kWideMid, kWideHalf, kWideQuarter, kWideShort, kWideTiny, kWidePair, kWideThin
};
// Estimated time (us) of a lone launch: the busiest CU runs c workgroups of U
// units per wave; a lone workgroup takes fix + lat U, bound by one wave's chain,
// and c of them base + c (thr U + o).  Fitted to 1378 measured products (1049 with
// per-group scales) of 5-16384 tokens, 64-14336 rows, 128-14336 weights a row, every
// shape timed on each.  On 689 (526) others its choice takes 1.004 (1.006) times
// the best shape's time on average, at most 1.19 (1.28).  (The constants before,
// fitted to fewer and larger products: 1.022 and 1.036, at most 1.29 and 1.49, and
// a few slower than on the kernel before these shapes: 261 x 10556 x 14208 63.8 ->
// 69.2 us.)
struct WideCost {
  int tokens, tiles, parts;
  float fix, lat, base, thr, o;
};
constexpr WideCost kWideCost[] = {
    {128, 4, 1, 9.127f, 0.68f, 5.442f, 0.558f, 3.541f},  // long
    {64, 4, 1, 6.417f, 0.651f, 3.916f, 0.368f, 2.424f},  // mid
    {64, 2, 2, 6.996f, 0.674f, 4.575f, 0.50f, 1.799f},   // half
    {64, 2, 4, 7.5f, 0.83f, 4.324f, 0.882f, 5.2f},       // quarter (eight waves)
    {32, 1, 4, 5.0f, 0.55f, 4.453f, 0.41f, 1.1f},        // short
    {32, 1, 8, 5.3f, 0.83f, 3.095f, 0.78f, 2.55f},       // tiny (eight waves)
    {32, 2, 2, 0, 0, 0, 0, 0},                           // pair (grouped launches)
    {32, 4, 1, 0, 0, 0, 0, 0},                           // thin (grouped launches)
};
// The shapes with per-group scales (long, quarter and thin are not offered).
constexpr WideCost kWideGroupCost[] = {
    {},
    {64, 4, 1, 4.905f, 0.952f, 2.233f, 0.604f, 2.635f},  // mid
    {64, 2, 2, 5.863f, 0.80f, 4.047f, 0.701f, 1.483f},   // half
    {},
    {32, 1, 4, 4.916f, 0.829f, 4.793f, 0.572f, 0.328f},  // short
    {32, 1, 8, 5.6f, 1.07f, 3.616f, 0.971f, 3.216f},     // tiny (eight waves)
    {32, 2, 2, 4.358f, 0.74f, 3.939f, 0.435f, 0.723f},   // pair
    {},
};
// `workgroups` of rows of `units` units; a part is whole chunks of `chunk` units.
constexpr float wide_estimate(const WideCost& c, int64_t workgroups, int64_t units,
                              int64_t chunk = 1) {
  const float u = static_cast<float>(ceil_div(ceil_div(units, c.parts), chunk) * chunk);
  const float per = static_cast<float>(ceil_div(workgroups, 256));
  const float one = c.fix + c.lat * u, many = c.base + per * (c.thr * u + c.o);
  return one > many ? one : many;
}
// The offer with the lowest estimate.
struct WidePick {
  int best = -1;
  float t = 0.0f;
  constexpr void offer(int shape, float e) {
    if (best < 0 || e < t) t = e, best = shape;
  }
};

// A lone product.
constexpr int wide_pick(int64_t m, int64_t n, int64_t k) {
  WidePick q{};
  for (int i : {kWideLong, kWideMid, kWideHalf, kWideQuarter, kWideShort, kWideTiny}) {
    const WideCost& c = kWideCost[i];
    q.offer(i, wide_estimate(c, ceil_div(ceil_div(n, 64), c.tiles) * ceil_div(m, c.tokens),
                             ceil_div(k, 128)));
  }
  return q.best;
}
// With per-group scales (pieces: read 16 bytes, four units, at a time).
constexpr int wide_pick_group(int64_t m, int64_t n, int64_t k, bool pieces) {
  WidePick q{};
  for (int i : {kWideMid, kWideHalf, kWidePair, kWideShort, kWideTiny}) {
    const WideCost& c = kWideGroupCost[i];
    q.offer(i, wide_estimate(c, ceil_div(ceil_div(n, 64), c.tiles) * ceil_div(m, c.tokens),
                             ceil_div(k, 128), pieces ? 4 : 1));
  }
  return q.best;
}

// Prepared blocks of a grouped launch: 8 tiles (4 with per-group scales) x 32
// tokens when the launch value is at most 32, else 8 tiles x 64 tokens.
constexpr int64_t wide_blocks(int64_t n, bool group_scales) {
  return ceil_div(ceil_div(n, 64), group_scales ? 4 : 8);
}
constexpr int wide_batched_tokens(int max_m) { return max_m <= 32 ? 32 : 64; }

// Shapes of the grouped launches.  A launch knows its blocks, its number of
// products and its longest m, not its products' rows: the lines are drawn for
// products of one row length (the projections of one input), and where a mix of
// lengths (1 to 112 units) would run far longer on the shape that is best for
// those, they give way.  Figures: mean time over the best shape's, products of one
// length / mixed, about 100 launches each.
//
// 8 x 64 blocks.  Up to 128 one round of the smaller shapes (33 .. 64: 64 x 2 1.00 /
// 1.45, 32 x 1 1.30 / 1.01; 65 .. 128: 64 x 4 1.06 / 1.8, 64 x 2 1.05 / 1.15, but up to
// 1.05 times the launch before these shapes; past that up to 1.3 times).  More: 64
// x 4 or 128 x 4 by rounds of workgroups at 24 units a row, an odd last token block
// priced for 128 x 4: one workgroup runs both halves of its tiles in series, 64
// tokens of each idle (129 .. 256 blocks: 128 x 4 1.53 / 2.9 with an odd one, 1.03 /
// 1.75 without; 64 x 4 1.00 / 1.5 and 1.03 / 1.45).
constexpr WideCost kGroupedLong{128, 4, 1, 8.2f, 0.68f, 5.0f, 0.64f, 7.7f};
constexpr WideCost kGroupedMid{64, 4, 1, 6.0f, 0.54f, 5.0f, 0.45f, 1.7f};
constexpr int64_t kWideUnits = 24;
constexpr int wide_pick_batched(int64_t total_blocks, int max_m) {
  if (total_blocks <= 128) return total_blocks <= 32 ? kWideShort : total_blocks <= 64 ? kWideHalf : kWideMid;
  const int64_t tb = ceil_div(max_m, 64);
  const float longs =
      wide_estimate(kGroupedLong, ceil_div(total_blocks * ((tb + 1) / 2 * 2), tb), kWideUnits) +
      (tb % 2 ? kGroupedLong.lat * kWideUnits : 0.0f);
  return longs <= wide_estimate(kGroupedMid, 2 * total_blocks, kWideUnits) ? kWideLong : kWideMid;
}
// 8 x 32 blocks.  65 .. 96: 32 x 1 1.18 / 1.00 (32 x 2 1.01 / 1.53); 97 .. 192: 32
// x 2 1.02 / 1.5 (32 x 1 1.4 / 1.00, and slower than the launch before these
// shapes); 193 and more: 32 x 4 1.00 (32 x 2 1.13 .. 1.27).
constexpr int wide_pick_batched32(int64_t total_blocks) {
  return total_blocks <= 96 ? kWideShort : total_blocks <= 192 ? kWidePair : kWideThin;
}
// 4 x 32 blocks of products with per-group scales.  Up to 128: 32 x 1 1.00 .. 1.05 /
// 1.00 (32 x 2 1.2 .. 1.02 / 1.4); 129 .. 384: 32 x 2 1.02 / 1.27 (32 x 1 1.2 ..
// 1.46 / 1.02, with one length up to 1.2 times the launch before these shapes);
// 385 .. 768: 32 x 2 1.13 / 1.06 (64 x 2 1.06 / 1.26, mixed up to 1.28 times the
// launch before; 64 x 4 1.01 .. 1.24 / 1.7); 769 .. 1536: 64 x 4 1.03 / 1.35 for the
// few projections of one input, 64 x 2 1.08 / 1.09 for more products; past that
// 64 x 4 1.01 / 1.15 (64 x 2 1.08 / 1.04).  The 64-token shapes take two blocks at a
// time, which launches of fewer than 32 tokens do not have: half of their work
// would be idle.
constexpr int wide_pick_batched_group(int64_t total_blocks, int count, int max_m) {
  if (total_blocks <= 128) return kWideShort;
  if (total_blocks <= 768 || max_m < 32) return kWidePair;
  return total_blocks <= 1536 && count > 3 ? kWideHalf : kWideMid;
}

// The block that workgroup b of a grid runs where workgroups that read the same
// data are neighbours.  Workgroups are dispatched to the 8 XCDs in turn (b -> XCD
// b % 8), each with its own L2; XCD x takes the x-th contiguous eighth of the
// blocks, so that the neighbours meet in few L2s and the data is fetched there
// once.
constexpr int xcd_block(int b, int grid) {
  constexpr int kXcds = 8;
  const int q = grid / kXcds, r = grid % kXcds;
  const int x = b % kXcds, slot = b / kXcds;
  return x < r ? x * (q + 1) + slot : r * (q + 1) + (x - r) * q + slot;
}

// Whether a lone product's workgroups (tile groups first) are taken so: products
// of few rows, whose activations outweigh their weights and were fetched by
// every XCD.  Time against the plain order, 256 .. 8192 tokens x 512 .. 14336
// weights a row: 320 rows 0.90 (6500 x 320 x 8192 47.5 -> 39.1 us), 640 0.92, 1024
// 0.93, 2048 0.97; 3072 1.01, 8192 1.03, 14336 1.04.
constexpr bool wide_xcd_order(int tiles) { return tiles <= 32; }

// What a workgroup of a grouped launch runs: tile groups g, g + step, ..
// (reps of them, one after the other; those past the tiles are left out) of the
// tokens from t0; reps = 0: nothing.
struct WideRun {
  int g, reps, step;
  int64_t t0;
  bool odd;  // an odd last token block, where the kernel has a shape for it
};

// Block lb of a product of R tiles and m tokens, part sub of its workgroups,
// each of `tiles` tiles.  8 x 64 blocks; with 128 tokens every two blocks of one
// tile group (an even and the next token block) are run by two workgroups of
// four tiles each.
constexpr WideRun wide_run64(int tokens, int tiles, int lb, int sub, int64_t m, int R) {
  const int gb = (R + 7) / 8;  // tile groups of a prepared block
  WideRun r{0, 1, 1, 0, false};
  if (tokens <= 64) {
    const int rpb = 8 / tiles;  // workgroups along the rows
    const int tb = lb / gb;
    r.t0 = int64_t(tb) * 64 + sub / rpb * tokens;
    r.g = (lb - tb * gb) * rpb + sub % rpb;
  } else {
    const int T = static_cast<int>((m + 63) / 64);
    const int pairs = T / 2 * 2 * gb;  // blocks of the paired token blocks
    const bool paired = lb < pairs;
    const int q = paired ? lb : 2 * (lb - pairs);  // the last, odd token block: both
    r.reps = paired ? 1 : 2;                       // halves of its tiles
    const int pr = paired ? q / (2 * gb) : T / 2;
    r.g = paired ? q - pr * 2 * gb : q;
    r.t0 = int64_t(pr) * 128;
  }
  if (r.t0 >= m) r.reps = 0;
  return r;
}

// 8 x 32 blocks, run by `per` workgroups each.
constexpr WideRun wide_run32(int tiles, int per, int lb, int sub, int64_t m, int R) {
  const int gb = (R + 7) / 8, tb = lb / gb, rpb = 8 / tiles;
  return {(lb - tb * gb) * rpb + sub, int64_t(tb) * 32 < m ? rpb / per : 0, per, int64_t(tb) * 32,
          false};
}

// 4 x 32 blocks of a product with per-group scales, run by `per` workgroups each.
// 64 tokens take two token blocks at a time: with four tiles the first half of a
// product's blocks run them, with two tiles each block takes half of the tiles.
// There an odd last token block is run block by block, by a 32 x 4 shape (both
// halves of its tiles in series took the launch up to 1.6 times as long).
constexpr WideRun wide_run32_group(int tokens, int tiles, int per, int lb, int sub, int64_t m,
                                   int R) {
  const int gb = (R + 3) / 4, tb = lb / gb;
  WideRun r{lb - tb * gb, 1, 1, int64_t(tb) * tokens, false};
  if (tokens == 32) {
    const int rpb = 4 / tiles;
    r = {r.g * rpb + sub, rpb / per, per, int64_t(tb) * 32, false};
  } else if (tiles == 2) {
    const int pairs = static_cast<int>((m + 31) / 64) * 2 * gb;  // blocks of the paired token blocks
    r.odd = lb >= pairs;
    r.g = r.odd ? lb - pairs : lb % (2 * gb);
    r.t0 = int64_t(lb / (2 * gb)) * 64;
  }
  if (r.t0 >= m) r.reps = 0;
  return r;
}

}  // namespace sherry
