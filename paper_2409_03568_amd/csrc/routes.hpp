// Which kernels take a call, where there is a choice: rules on sizes, with the timings that they
// follow.  Plain host code without device types, so that they can be tested anywhere.
#pragma once
#include <stdint.h>

namespace ckks {

// Encryption splits a pixel's rows over workgroups (k_encrypt_few) up to this many pixels per 4
// CUs: see RingLaunch::encrypt_as.
constexpr uint64_t few_per_4_cus(int log_n) { return log_n == 11 ? 1 : log_n == 13 ? 4 : 2; }

// How the misses of a batch (every pixel without a cache) are encrypted and decrypted: by the
// batch's persistent launch (k_cached_fused), which does with one workgroup's share of the ring and
// no launch of its own, or apart, by the kernels of plain encryption and decryption, a pair of
// launches for each ring of ciphertexts.  The pairs' transforms are cheaper, but each pair fills and
// drains the device, and with a cache all pairs that could be needed are launched, whatever it
// misses.  Where the number of misses decides, kCounted, the device chooses: apart from half a
// wave of workgroups of them on.  In ms, persistent / apart:
//   no cache     N = 2048: 5,000 pixels, ring 8192: .39 / .36;  30,000, ring 2048: 1.94 / 2.12, 8192: 1.96 / 1.92
//                N = 4096: 30,000, ring 64: 20.3 / 18.1, 512: 4.06 / 6.58, 2048: 4.07 / 4.10, 4096: 4.10 / 4.07
//                N = 8192: 30,000, ring 64: 50.3 / 28.0, 256: 12.8 / 14.0, 512: 12.8 / 10.8, 8192: 12.8 / 9.7
//                N = 16384: 5,000, ring 64: 37.1 / 11.5, 8192: 10.3 / 6.1
//                one ring for all: 300 pixels .10 / .07, .13 / .10, .25 / .20 and 1.03 / .60
//   top-k cache  N = 2048: 30,000, ring 8192: 1.58 / 1.67 with 3 in 4 missing, .82 / .90 with 1 in 40
//                N = 4096: 5,000, ring 8192: .60 / .64 and .36 / .43;  30,000: 3.37 / 3.31 and 1.64 / 1.66
//                N = 8192: 30,000, ring 256: 10.5 / 11.6 and 4.6 / 5.3, ring 512: 10.5 / 9.1 and 4.6 / 4.5;
//                          1,000 and 2,000 pixels, ring 8192: .44 / .45 and .77 / .67 with 3 in 4 missing,
//                          .23 / .25 and .47 / .53 with 1 in 40
//                N = 16384: 30 .. 50% apart at every ring and count
enum BatchRoute : int { kFused = 0, kApart = 1, kCounted = 2 };
constexpr uint64_t kMaxMissPairs = 1024;  // bounds the launches, and a captured graph, whatever the batch
inline BatchRoute batch_route(int log_n, bool cached, uint64_t n, uint64_t ring, uint64_t cus) {
  if (n > ring * kMaxMissPairs) return kFused;
  if (log_n == 14) return kApart;
  if (cached) return log_n == 13 && ring >= 2 * cus && n >= 6 * cus ? kCounted : kFused;
  if (ring >= n) return kApart;
  if (log_n > 11 && 2 * ring <= cus) return kApart;  // their pixels are split over workgroups
  return ring >= (log_n == 11 ? 32 : log_n == 12 ? 16 : 2) * cus ? kApart : kFused;
}

}  // namespace ckks
