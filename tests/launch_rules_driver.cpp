// Answers of the launch rules on the CPU: one query per line of stdin (a name
// and integers), one line of integers per answer.
#include <cstdio>
#include <iostream>
#include <sstream>
#include <string>
#include <vector>

#include "launch_rules.h"

using namespace sherry;

namespace {

// Runs every workgroup of a grouped launch of products (m, R tiles) on one
// shape.  kind 64: 8 x 64 blocks; 32: 8 x 32 blocks; 33: 4 x 32 blocks of products
// with per-group scales.  Prints the (tile, token) cells not run exactly once,
// the most tile groups that one workgroup runs in series, and the workgroups
// with work.
void cover(const std::vector<int64_t>& a) {
  const int kind = static_cast<int>(a[0]), per = static_cast<int>(a[2]);
  const WideCost c = (kind == 33 ? kWideGroupCost : kWideCost)[a[1]];
  struct Product {
    int m, R, begin, count;
    std::vector<int> runs;  // [R][m]
  };
  std::vector<Product> ps;
  int total = 0;
  for (size_t i = 3; i + 1 < a.size(); i += 2) {
    Product p{static_cast<int>(a[i]), static_cast<int>(a[i + 1]), total, 0, {}};
    p.count = static_cast<int>(wide_blocks(int64_t(p.R) * 64, kind == 33) *
                               ceil_div(p.m, kind == 64 ? 64 : 32));
    p.runs.assign(size_t(p.R) * p.m, 0);
    total += p.count;
    ps.push_back(p);
  }
  int series = 0, active = 0;
  for (int b = 0; b < total * per; ++b) {
    const int blk = b / per;
    for (Product& p : ps) {
      if (blk < p.begin || blk >= p.begin + p.count) continue;
      const WideRun r =
          kind == 64 ? wide_run64(c.tokens, c.tiles, blk - p.begin, b % per, p.m, p.R)
          : kind == 32 ? wide_run32(c.tiles, per, blk - p.begin, b % per, p.m, p.R)
                       : wide_run32_group(c.tokens, c.tiles, per, blk - p.begin, b % per, p.m,
                                          p.R);
      const bool thin = r.odd && c.tiles == 2;  // (the kernel's 32 x 4 shape)
      const int tokens = thin ? 32 : c.tokens, tiles = thin ? 4 : c.tiles;
      int done = 0;
      for (int h = 0; h < r.reps; ++h) {
        const int g = r.g + h * r.step;
        if (g * tiles >= p.R) break;
        ++done;
        for (int t = g * tiles; t < (g + 1) * tiles && t < p.R; ++t)
          for (int64_t m = r.t0; m < r.t0 + tokens && m < p.m; ++m) ++p.runs[size_t(t) * p.m + m];
      }
      if (done > series) series = done;
      active += done > 0;
    }
  }
  int bad = 0;
  for (const Product& p : ps)
    for (int n : p.runs) bad += n != 1;
  std::printf("%d %d %d\n", bad, series, active);
}

}  // namespace

int main() {
  std::string line;
  while (std::getline(std::cin, line)) {
    std::istringstream in(line);
    std::string fn;
    in >> fn;
    std::vector<int64_t> a;
    for (int64_t v; in >> v;) a.push_back(v);
    if (fn == "quant_streams") {
      std::printf("%d\n", quant_streams(a[0], a[1]) ? 1 : 0);
    } else if (fn == "quant_shape") {
      const QuantShape q = quant_shape(a[0], a[1]);
      std::printf("%d %d\n", q.threads, q.pieces);
    } else if (fn == "sm_splits") {
      std::printf("%d\n", a[1] <= kSmFoldBlocks && sm_splits(a[0], a[1], a[2] != 0) ? 1 : 0);
    } else if (fn == "sm_whole_sub") {
      std::printf("%d\n", sm_whole_sub(static_cast<int>(a[0])));
    } else if (fn == "xcd_block") {
      for (int b = 0; b < a[0]; ++b) std::printf("%d ", xcd_block(b, static_cast<int>(a[0])));
      std::printf("\n");
    } else if (fn == "wide_pick") {
      std::printf("%d\n", wide_pick(a[0], a[1], a[2]));
    } else if (fn == "wide_pick_group") {
      std::printf("%d\n", wide_pick_group(a[0], a[1], a[2], a[3] != 0));
    } else if (fn == "wide_pick_batched") {
      std::printf("%d\n", wide_pick_batched(a[0], static_cast<int>(a[1])));
    } else if (fn == "wide_pick_batched32") {
      std::printf("%d\n", wide_pick_batched32(a[0]));
    } else if (fn == "wide_pick_batched_group") {
      std::printf("%d\n", wide_pick_batched_group(a[0], static_cast<int>(a[1]), static_cast<int>(a[2])));
    } else if (fn == "cover") {
      cover(a);
    } else {
      std::fprintf(stderr, "unknown query: %s\n", fn.c_str());
      return 1;
    }
  }
  return 0;
}
