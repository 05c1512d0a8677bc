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

static void encryption() {
  for (uint64_t cus : {64ull, 256ull, 304ull})
    for (int log_n = 11; log_n <= 14; log_n++)
      for (int primes = 1; primes <= 16; primes++)
        for (uint64_t n = 1; n < 100000; n += n < 5000 ? 1 : 997) {
          const EncKernel k = encrypt_kernel(log_n, primes, n, cus);
          if (k == kEncSplit) CHECK(n <= cus);       // parts of at least one workgroup per CU
          if (k == kEncPrime) CHECK(log_n <= 13);    // the kernels that are compiled
          // a single prime leaves the complex transforms nothing to share at small rings
          if (log_n <= 12 && primes == 1) CHECK(k == kEncPrime);
          // at N = 8192 a round that leaves CUs part empty takes the prime-field kernel
          if (log_n == 13 && primes < 8 && 3 * n > 2 * cus && n <= cus) CHECK(k == kEncPrime);
          if (log_n == 13 && primes > 1 && n > cus) CHECK(k == kEncComplex);
        }
  CHECK(encrypt_kernel(12, 3, 700, 256) == kEncPrime);
  CHECK(encrypt_kernel(12, 3, 1024, 256) == kEncComplex);
  CHECK(encrypt_kernel(12, 3, 1500, 256) == kEncPrime);
  CHECK(encrypt_kernel(12, 3, 65536, 256) == kEncComplex);
  CHECK(encrypt_kernel(11, 8, 1000, 256) == kEncPrime);
  CHECK(encrypt_kernel(11, 8, 2048, 256) == kEncComplex);
  CHECK(encrypt_kernel(13, 2, 200, 256) == kEncPrime);
  CHECK(encrypt_kernel(13, 4, 129, 256) == kEncSplit);
  CHECK(encrypt_kernel(13, 12, 256, 256) == kEncSplit);
}

static void decryption() {
  for (int log_n : {11, 12, 14}) CHECK(!decrypt_complex(log_n, 1, 2, 1000000, 256));
  // few ciphertexts, and one limb up to several rounds of workgroups, take the prime-field kernel
  for (uint64_t n : {1ull, 256ull}) CHECK(!decrypt_complex(13, 1, 2, n, 256));
  for (uint64_t n : {300ull, 700ull, 2000ull}) CHECK(!decrypt_complex(13, 1, 1, n, 256) && !decrypt_complex(13, 0, 1, n, 256));
  CHECK(!decrypt_complex(13, 0, 2, 511, 256));
  CHECK(decrypt_complex(13, 1, 2, 300, 256) && decrypt_complex(13, 0, 2, 1000, 256));
  CHECK(decrypt_complex(13, 1, 1, 8000, 256) && decrypt_complex(13, 0, 1, 10000, 256));
}

static void cached_misses() {
  for (bool beside : {false, true})
    for (int log_n = 11; log_n <= 14; log_n++)
      for (int primes = 1; primes <= 16; primes++)
        for (uint64_t n : {1ull, 128ull, 129ull, 200ull, 240ull, 256ull, 289ull, 512ull, 1024ull, 1025ull, 4000ull, 65536ull}) {
          const MissRoute r = miss_route(log_n, primes, beside, n, 256);
          const bool asked = r.few_below || r.few_share;
          if (log_n == 14) CHECK(!asked && r.many < 0);  // kernels that are compiled
          if (asked) CHECK(n > (log_n == 13 ? 256 : 1024) && log_n < 14);
          // complex encryptions of the whole device beside the gather only for many misses
          if (asked && beside) CHECK(r.few != kEncComplex || r.few_grid == 256);
          // after it few take the kernel of the lower latency
          if (asked && !beside) CHECK(r.few == kEncPrime && r.many == kEncComplex);
          // up to two pixels per CU as many misses as there are CUs or fewer take the prime-field
          // kernel, in one round, and more the complex one where there are primes to share
          if (log_n < 13 && n > 256 && n <= 512) CHECK(!asked && r.many == kEncPrime);
          if (log_n == 13 && n > 256 && n <= 512) {
            CHECK(r.few == kEncPrime && (!asked || r.few_below == 257));
            CHECK(r.many == (primes > (beside ? 1 : 2) ? kEncComplex : kEncPrime));
          }
          if (log_n == 11 && n > 256 && (beside || primes < 8)) CHECK(r.many == kEncPrime);
          // a short list: one launch, on either stream alike; the prime-field kernel, which takes
          // longest for a single miss, only where it has few primes or a pixel for every CU
          if (n > 256) continue;
          CHECK(!asked && r.few == r.many);
          const int kernel = r.many < 0 ? encrypt_kernel(log_n, primes, n, 256) : r.many;
          if (log_n == 13 && primes > 2 && n <= 170) CHECK(kernel == kEncSplit);
          if (log_n == 13 && primes > 3 && n <= 240) CHECK(kernel == kEncSplit);
          if (log_n == 13 && primes < 3 && n > 128) CHECK(kernel == kEncPrime);
        }
}

int main() {
  decryption();
  cached_misses();
  batches();
  encryption();
  if (!failures) printf("ok\n");
  return failures != 0;
}
