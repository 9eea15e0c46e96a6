// A batched call's worker contexts describe the caller's device: with the compute units of another
// device than the default one, and every setting that worker_of copies away from its default.
#include <cstdio>

#include "internal.h"

int main() {
  int fail = 0;
  auto check = [&](bool ok, const char *what) {
    if (!ok) std::fprintf(stderr, "FAIL: %s\n", what), ++fail;
  };
  dacp_ctx_s a, b;
  a.device = 3;
  a.num_cus = 32;
  a.batch_workers = 2;
  a.tile_elems = 512;
  a.two_pass_min_L = 11;
  a.dc_min_n = 7;
  a.blocked_min_n = 900;
  a.tri_spins = 12;
  a.red_elems = 5;
  b.worker_of(a);
  check(b.device == 3, "device");
  check(b.num_cus == 32, "compute units");
  check(b.batch_workers == 2, "host threads");
  check(b.tile_elems == 512 && b.two_pass_min_L == 11 && b.dc_min_n == 7 && b.blocked_min_n == 900 && b.tri_spins == 12, "knobs");
  check(b.red == nullptr && b.red_elems == 0 && b.stream == nullptr, "a worker's own buffers and stream");
  std::printf("%d failures\n", fail);
  return fail != 0;
}
