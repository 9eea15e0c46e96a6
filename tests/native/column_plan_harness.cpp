// Column groups of the memory recurrences: every column exactly once, no launch past the cache, and padding only
// where it is the faster way (times of 9 to 33 columns of a chain on MI355X).
#include <cstdio>
#include <initializer_list>

#include "host_rules.h"

using dacp::rules::ColumnPlan;
using dacp::rules::column_plan;

int main() {
  int fail = 0;
  auto check = [&](bool ok, const char *what, int L, int b) {
    if (!ok) std::fprintf(stderr, "FAIL: %s (L %d, b %d)\n", what, L, b), ++fail;
  };
  auto from = [](int least) { return [least](int w) { return w >= least && (w & (w - 1)) == 0; }; };
  // columns that all launches together advance, the padding included
  auto advanced = [](const ColumnPlan &p, int b) {
    return p.fused ? (b - p.tail + p.g - 1) / p.g * p.g + p.tail_w : b;
  };
  for (int L = 15; L <= 24; ++L)
    for (int b = 1; b <= 130; ++b)
      for (int g : {1, 2, 3, 5, 8, 16})
        for (int least : {2, 4, 64})
          for (bool filter : {false, true}) {
            const int gw = g < b ? g : b;
            const int64_t D = int64_t(1) << L, bytes = 24 + 8 * filter;
            const ColumnPlan p = column_plan(D, b, gw, bytes, least == 4, filter, from(least));
            check(p.g >= gw && p.per >= 1 && p.tail >= 0 && p.tail < b, "sizes", L, b);
            check(p.tail == 0 || (p.fused && p.tail_w >= p.tail && p.tail_w < p.g && (b - p.tail) % p.g == 0), "tail", L, b);
            check(p.per == 1 || D * p.g * p.per * bytes <= dacp::rules::kRecCacheBytes, "cache", L, b);
          }
  auto evolution = [&](int L, int b) { return column_plan(int64_t(1) << L, b, b < 8 ? b : 8, 24, false, false, from(2)); };
  auto filtered = [&](int L, int b, bool mixed) {
    return column_plan(int64_t(1) << L, b, b < 8 ? b : 8, 32, mixed, true, from(mixed ? 4 : 2));
  };
  for (int b : {9, 10, 12, 17, 25, 33}) {  // one padded group too many cost 10 to 26 % at 2^20 rows
    check(advanced(evolution(20, b), b) <= b + 1, "evolution, 2^20 rows", 20, b);
    check(advanced(filtered(20, b, false), b) <= b + 1, "filter, 2^20 rows", 20, b);
    check(advanced(filtered(20, b, true), b) <= b + 1, "mixed filter, 2^20 rows", 20, b);
    check(advanced(filtered(19, b, false), b) <= b + 1, "filter, 2^19 rows", 19, b);
  }
  for (int b : {9, 10, 17}) check(advanced(evolution(18, b), b) <= b + 1, "evolution, 2^18 rows", 18, b);
  for (int b : {9, 12, 23}) {  // together in one launch where launches are what a step costs
    check(evolution(15, b).tail == 0 && evolution(15, b).per == (b + 7) / 8, "one launch", 15, b);
    check(filtered(18, b, false).tail == 0, "filter, 2^18 rows", 18, b);
    check(filtered(19, b, true).tail == 0 || b == 23, "mixed filter, 2^19 rows", 19, b);
  }
  check(advanced(evolution(20, 13), 13) == 16, "five columns left are a group", 20, 13);
  check(!filtered(16, 5, true).fused && filtered(16, 8, true).fused && filtered(17, 5, true).fused, "small mixed", 16, 5);
  std::printf("%d failures\n", fail);
  return fail != 0;
}
