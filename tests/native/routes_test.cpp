// Host test of the rules that choose kernels (routes.hpp).
#include <initializer_list>

#include <stdint.h>
#include <stdio.h>

#include "../../paper_2409_03568_amd/csrc/routes.hpp"

using namespace ckks;

static int failures = 0;
#define CHECK(cond)                                            \
  do {                                                         \
    if (!(cond)) {                                             \
      printf("line %d: %s\n", __LINE__, #cond);                \
      failures++;                                              \
    }                                                          \
  } while (0)

// Pairs of launches for the misses of a batch (0: none beside the persistent launch).
static uint64_t pairs(int log_n, bool cached, uint64_t n, uint64_t ring, uint64_t cus) {
  return batch_route(log_n, cached, n, ring, cus) != kFused ? (n + ring - 1) / ring : 0;
}

static void batches() {
  for (uint64_t cus : {64ull, 256ull, 304ull})
    for (int log_n = 11; log_n <= 14; log_n++)
      for (uint64_t ring : {1ull, 2ull, 64ull, 100ull, 256ull, 511ull, 512ull, 4096ull, 8192ull, 100000ull})
        for (uint64_t n : {1ull, 64ull, 100ull, 1025ull, 65536ull, 5500000ull, 4000000000ull})
          for (bool cached : {false, true}) {
            // launches stay bounded whatever the batch
            CHECK(pairs(log_n, cached, n, ring, cus) <= 1024);
            // a cached batch launches for misses that may not be there only where that pays
            if (cached && log_n <= 12) CHECK(pairs(log_n, cached, n, ring, cus) == 0);
            if (cached && log_n == 13 && ring < 2 * cus) CHECK(pairs(log_n, cached, n, ring, cus) == 0);
            // without a cache every pixel misses: nothing to count
            if (!cached || log_n != 13) CHECK(batch_route(log_n, cached, n, ring, cus) != kCounted);
          }
  CHECK(batch_route(13, false, 65536, 8192, 256) == kApart);
  CHECK(batch_route(13, true, 65536, 8192, 256) == kCounted);
  CHECK(batch_route(13, true, 300, 8192, 256) == kFused);
  CHECK(batch_route(14, true, 300, 64, 256) == kApart);
  CHECK(batch_route(12, false, 300, 8192, 256) == kApart);
  CHECK(batch_route(11, false, 30000, 2048, 256) == kFused);
  CHECK(batch_route(12, false, 30000, 512, 256) == kFused);
  CHECK(batch_route(13, false, 30000, 256, 256) == kFused);
  CHECK(batch_route(13, false, 30000, 64, 256) == kApart);
}

int main() {
  batches();
  if (!failures) printf("ok\n");
  return failures != 0;
}
