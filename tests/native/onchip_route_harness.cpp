// The on-chip route's rule against what both routes took on MI355X (microseconds an apply, FP64 filter): the
// chosen one is never more than 15 % above the faster one.
#include <algorithm>
#include <cstdio>

#include "host_rules.h"

struct Row {
  int L, flips, masks, plain, sign, b;
  double onchip, memory;
};

static const Row kRows[] = {
    // chain: L single-spin flips
    {8, 8, 8, 0, 0, 1, 0.6, 3.5}, {10, 10, 10, 0, 0, 64, 0.8, 6.1}, {12, 12, 12, 0, 0, 8, 1.9, 5.8}, {13, 13, 13, 0, 0, 2, 3.0, 6.0},
    {14, 14, 14, 0, 0, 1, 5.66, 6.02}, {14, 14, 14, 0, 0, 16, 5.8, 8.7}, {14, 14, 14, 0, 0, 64, 6.0, 13.2}, {14, 14, 14, 0, 0, 256, 6.3, 47.3},
    // nearest-neighbour pairs: L - 1
    {11, 10, 10, 10, 0, 1, 1.5, 5.1}, {12, 11, 11, 11, 0, 32, 2.5, 6.8}, {13, 12, 12, 12, 0, 1, 4.47, 5.98}, {13, 12, 12, 12, 0, 64, 4.7, 10.5},
    {14, 13, 13, 13, 0, 1, 8.8, 6.46}, {14, 13, 13, 13, 0, 2, 8.8, 6.21}, {14, 13, 13, 13, 0, 8, 8.85, 7.12}, {14, 13, 13, 13, 0, 16, 9.0, 8.89},
    {14, 13, 13, 13, 0, 32, 9.1, 10.6}, {14, 13, 13, 13, 0, 64, 9.04, 13.0}, {14, 13, 13, 13, 0, 256, 9.4, 45.5},
    // all pairs: L (L - 1) / 2
    {10, 45, 45, 45, 0, 1, 3.3, 10.4}, {11, 55, 55, 55, 0, 8, 5.0, 14.7}, {12, 66, 66, 66, 0, 1, 9.2, 15.6}, {12, 66, 66, 66, 0, 64, 9.4, 19.1},
    {13, 78, 78, 78, 0, 1, 20.5, 18.7}, {13, 78, 78, 78, 0, 16, 20.5, 20.3}, {13, 78, 78, 78, 0, 64, 21.0, 26.6}, {13, 78, 78, 78, 0, 256, 21.2, 86.9},
    {14, 91, 91, 91, 0, 1, 46.7, 21.1}, {14, 91, 91, 91, 0, 8, 46.7, 22.7}, {14, 91, 91, 91, 0, 16, 46.8, 24.0}, {14, 91, 91, 91, 0, 32, 47.0, 29.7},
    {14, 91, 91, 91, 0, 64, 47.3, 50.9}, {14, 91, 91, 91, 0, 128, 47.4, 96.7}, {14, 91, 91, 91, 0, 256, 47.5, 191.4},
    // nearest-neighbour pairs of both kinds, half of the flips with a sign
    {10, 18, 9, 9, 9, 1, 1.9, 6.5}, {12, 22, 11, 11, 11, 16, 4.6, 8.35}, {13, 24, 12, 12, 12, 1, 9.2, 8.5},
    {13, 24, 12, 12, 12, 32, 9.35, 11.2}, {14, 26, 13, 13, 13, 2, 19.8, 8.9}, {14, 26, 13, 13, 13, 32, 19.8, 13.3},
    {14, 26, 13, 13, 13, 64, 19.84, 18.4}, {14, 26, 13, 13, 13, 256, 20.15, 62.5},
    // all pairs of both kinds
    {12, 132, 66, 66, 66, 1, 21.9, 29.9}, {13, 156, 78, 78, 78, 2, 52, 35.1}, {13, 156, 78, 78, 78, 64, 52.5, 45.4},
    {13, 156, 78, 78, 78, 256, 52.9, 155.6}, {14, 182, 91, 91, 91, 16, 124, 43.2}, {14, 182, 91, 91, 91, 64, 124, 91},
    {14, 182, 91, 91, 91, 256, 124.6, 342.7},
};

int main() {
  int fail = 0;
  for (const Row &r : kRows) {
    const bool chip = dacp::rules::onchip_pays(r.L, {r.flips, r.masks, r.plain, r.sign}, r.b, 256, 1000, 0.0);
    const double took = chip ? r.onchip : r.memory;
    if (took > 1.15 * std::min(r.onchip, r.memory)) {
      std::fprintf(stderr, "FAIL: L %d flips %d b %d: %s\n", r.L, r.flips, r.b, chip ? "on chip" : "memory");
      ++fail;
    }
  }
  auto check = [&](bool ok, const char *what) {
    if (!ok) std::fprintf(stderr, "FAIL: %s\n", what), ++fail;
  };
  using dacp::rules::onchip_pays;
  const dacp::rules::FlipCounts chain{14, 14, 0, 0}, pairs{91, 91, 91, 0}, small{10, 10, 0, 0};
  check(onchip_pays(14, chain, 512, 256, 1000, 0.0), "two columns a compute unit");
  check(!onchip_pays(14, chain, 64, 1, 1000, 0.0), "64 columns on one compute unit");
  check(!onchip_pays(14, chain, 8, 256, 1e6, 0.0), "six seconds in one launch");
  check(!onchip_pays(14, pairs, 256, 256, 1e5, 0.0), "five seconds in one launch");
  check(onchip_pays(10, small, 8, 256, 1e6, 0.0), "under a second in one launch");
  std::printf("%d failures\n", fail);
  return fail != 0;
}
