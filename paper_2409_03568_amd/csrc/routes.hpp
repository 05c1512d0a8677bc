// Which kernels take a call, where there is a choice: rules on sizes, with the timings that they
// follow.  Plain host code without device types, so that they can be tested anywhere.
#pragma once
#include <stdint.h>

namespace ckks {

// Which kernel encrypts n pixels (of a list: by its capacity): a pixel's rows split over workgroups
// (k_encrypt_few), whole ciphertexts through prime-field transforms (k_encrypt_ntt, N <= 8192) or
// through complex ones (k_encrypt).  The complex transforms take less work from two or three primes
// on, where their one transform of v serves all, but a workgroup of theirs has a quarter of the
// threads, so a round of workgroups that leaves CUs part empty wants the prime-field ones.  In us,
// split / prime-field / complex, for n pixels on 256 CUs:
//   N = 2048, 1 prime:    64: 33 / 31 / 57   2,048: - / 66 / 74     10,240: - / 234 / 276
//             3 primes:   64: 39 / 41 / 82   2,560: - / 145 / 173   10,240: - / 516 / 505
//             4 primes:  128: 54 / 47 / 94   2,048: - / 149 / 144    3,072: - / 209 / 214   8,192: - / 529 / 494
//             8 primes:   64: 53 / 69 / 144  1,536: - / 207 / 216    2,560: - / 320 / 339   3,072: - / 391 / 352
//   N = 4096, 1 prime:   128: 38 / 36 / 60   4,096: - / 210 / 253   16,384: - / 778 / 863
//             2 primes:  128: 47 / 45 / 74   6,144: - / 495 / 493   10,240: - / 814 / 788
//             3 primes:  128: 55 / 55 / 88     768: - / 108 / 114    1,024: - / 132 / 125   1,536: - / 182 / 214
//                      2,560: - / 294 / 308  4,096: - / 450 / 438    8,192: - / 904 / 833
//             8 primes:  512: - / 168 / 215    768: - / 233 / 222    1,500: - / 412 / 430   2,560: - / 690 / 637
//   N = 8192, 1 prime:   192: 67 / 50 / 66     512: - / 84 / 80        768: - / 114 / 118   1,536: - / 204 / 197
//             4 primes:  128: 84 / 106 / 118   192: 118 / 108 / 118    256: 119 / 112 / 119   512: - / 202 / 165
//            16 primes:  192: 315 / 337 / 339  256: 320 / 350 / 342    512: - / 711 / 513
//   N = 16384, 4 primes: 128: 195 / - / 283    192: 310 / - / 288
enum EncKernel : int { kEncSplit = 0, kEncPrime = 1, kEncComplex = 2 };
inline EncKernel encrypt_kernel(int log_n, int primes, uint64_t n, uint64_t cus) {
  if (log_n == 14) return 2 * n <= cus ? kEncSplit : kEncComplex;
  if (log_n == 13) {
    if (2 * n <= cus || (primes > 2 && 3 * n <= 2 * cus) || (primes >= 8 && n <= cus)) return kEncSplit;
    if (n <= cus) return kEncPrime;
  } else if (primes > 1 && (log_n == 11 ? 4 : 2) * n <= cus) {
    return kEncSplit;
  }
  // complex from `from` pixels per CU on, and before that where the last round of as many
  // ciphertexts as the device holds is filled beyond `last` per CU (0: never)
  constexpr uint64_t kNever = ~0ull;
  uint64_t from, last;
  if (log_n == 11) {
    from = primes < 3 ? kNever : primes < 8 ? 32 : 12;
    last = primes < 4 ? 0 : 6;
  } else if (log_n == 12) {
    from = primes < 2 ? kNever : primes < 3 ? 32 : primes < 8 ? 20 : 8;
    last = primes < 3 ? 0 : primes < 8 ? 3 : 2;
  } else {
    from = primes < 2 ? 5 : 1;
    last = 1;
  }
  const uint64_t round = (uint64_t)(1 << (14 - log_n)) * cus;  // ciphertexts on the device at once
  if (from != kNever && n >= from * cus) return kEncComplex;
  return last && (n - 1) % round + 1 > last * cus ? kEncComplex : kEncPrime;
}

// Whether n ciphertexts are decrypted through complex transforms (else through prime-field ones).
// They win where there are many ciphertexts of N = 8192, and earlier for two limbs and for primes
// of more than 40 bits (prime_class 1), whose prime-field transforms need more reductions.  In
// us, prime-field / complex:
//   50 bits, one limb   300: 43.7 / 45.7   2,000: 122 / 126   3,000: 178 / 178   8,000: 448 / 420
//            two limbs  200: 35 / 37       300: 77.7 / 74.1   2,000: 264 / 238   8,000: 982 / 832
//   36 bits, one limb   300: 42.9 / 45.7   2,000: 117 / 125   5,000: 267 / 273   8,000: 417 / 416
//            two limbs  300: 74.5 / 74.2   511: 77.2 / 78.5   1,000: 136 / 134   8,000: 933 / 831
// At N = 4096 the complex ones win only for many ciphertexts (3.08 against 3.12 ms per 65,536, 173
// against 159 us for 3,200); at N = 2048, whose smaller primes need fewer reductions, they lose
// (1.43 against 1.36 ms), and at 2^14, whose 128 KB exchange space leaves one workgroup of 8 waves
// on a CU, too (20.7 against 16.9 ms).
inline bool decrypt_complex(int log_n, int prime_class, int limbs, uint64_t n, uint64_t cus) {
  const uint64_t per_cu = limbs == 2 ? (prime_class ? 1 : 3) : prime_class ? 16 : 32;
  return log_n == 13 && n > per_cu * cus;
}

// How the misses of a value cache among n pixels are encrypted: beside the gather of the hits on
// another stream, or after it.  Complex encryptions fill a CU's registers, so where they come first
// they hold up a gather beside them, and alone they have the longer latency while they are few: few
// misses take fewer workgroups or the prime-field kernel, many the whole device.  Which it
// is the device decides, by the misses being below `few_below` plus one in `few_share` of the hits
// (both 0: not asked, `many` takes any).  few_grid: workgroups (0: as for many).
// Beside the gather, in us, misses being 1 in 6 / 1 in 3 or 2 in 5 / 3 in 4 of the pixels:
//   N = 2048, 10,000 pixels: prime-field, 1 per CU 302 / 441 / 741, 2 per CU 312 / 323 / 523,
//                            unbounded 369 / 347 / 445; complex 418 / 433 / 481
//             65,536 pixels: prime-field, 1 per CU 1422 / 2580 / 4478, 2 per CU 1318 / 1944 / 3164,
//                            unbounded 1558 / 1780 / 2767; complex 1351 / 1827 / 2672
//   N = 4096, 10,000 pixels: prime-field, 1 per CU 510 / 677 / 1072, unbounded 481 / 586 / 895;
//                            complex 764 / 811 / 865
//   N = 8192, 10,000 pixels: prime-field, 1 per CU 1312 / 1739 / 2971; complex, 1 per CU
//                            1132 / 1679 / 2934, unbounded 1582 / 1625 / 2380
//             65,536 pixels: complex, 1 per CU 7025 / 11883 / 19574, unbounded 6761 / 10037 / 14817
//   1,024 pixels, prime-field unbounded against complex: N = 2048 109 / 112 / 123 against 144 / 142 / 148,
//   N = 4096 134 / 137 / 169 against 148 / 163 / 191, N = 8192 217 / 270 / 357 against 206 / 224 / 310
//   N = 8192, 1 per CU / unbounded, by primes:
//             1,200 pixels, 1 in 5 missing, 4: 210 / 214, 3 in 10: 283 / 229
//             1,500 pixels, 1 in 5, 1: 164 / 138, 2: 205 / 171, 4: 286 / 251; 3 in 10, 4: 291 / 350, 8: 615 / 645
//             2,000 pixels, 1 in 5, 4: 297 / 331, 3 in 10: 394 / 443;  3,000: 405 / 587, 501 / 617
//             12,000 pixels, 1 in 5, 1: 540 / 517, 2: 782 / 901; 3 in 10, 1: 751 / 621, 2: 1055 / 965
//             30,000 pixels, 1 in 5, 1: 1295 / 1145, 2: 1995 / 1887; 3 in 10, 1: 1802 / 1437, 4: 4976 / 4080
//   N = 2048, 8 primes, 1 per CU / 2, 3 in 10: 1,200 pixels 187 / 161, 8,000: 603 / 548, 12,000: 867 / 812
// Up to two pixels per CU at N = 8192, prime-field / complex by the count, 1 in 5 missing / all: beside
// the gather, 2 primes, 400 pixels 115 / 125, 173 / 162, 4 primes 154 / 164, 249 / 219; after it, 2
// primes 129 / 140, 170 / 168, 4 primes 181 / 194, 248 / 222, 8 primes 290 / 300, 410 / 334.
// After it, prime-field / complex, 1 in 6 missing: N = 4096, 1,000 pixels 181 / 214; N = 8192, 300
// pixels 181 / 193, 1,000 pixels 282 / 292.  With 8 primes, nearly all or all missing: N = 4096, 3,000
// pixels 961 / 890, N = 2048, 12,000 pixels 1727 / 1418 (3 in 10 992 / 977).
// Lists of no more than a pixel per CU go by their length, but one of four primes or more at N =
// 8192 is split over workgroups for longer than plain pixels are: workgroups without a miss leave
// at once, so that few misses have the device, and only lists that fill its last parts lose by it.
// Split / prime-field with 1 in 20 / 1 in 3 / all missing, after the gather, in us:
//   3 primes, 140 pixels 109 / 128, 120 / 125, 106 / 110;  200: 126 / 134, 137 / 130, 128 / 119
//   4 primes, 140 pixels 126 / 153, 137 / 151, 121 / 130;  234: 148 / 164, 162 / 158, 147 / 144;
//             256: 173 / 168, 165 / 160, 148 / 147
//   6 primes, 140 pixels 149 / 204, 167 / 201, 139 / 168;  234: 185 / 217, 207 / 209, 180 / 183
struct MissRoute {
  uint32_t few_below, few_share;
  int few, many;      // EncKernel, -1: by n
  uint64_t few_grid;
};
inline MissRoute miss_route(int log_n, int primes, bool beside, uint64_t n, uint64_t cus) {
  constexpr MissRoute by_n{0, 0, -1, -1, 0}, prime{0, 0, kEncPrime, kEncPrime, 0}, split{0, 0, kEncSplit, kEncSplit, 0};
  if (log_n == 13 && primes > 3 && 16 * n <= 15 * cus) return split;
  if (log_n == 14 || n <= cus) return by_n;
  const MissRoute counted{(uint32_t)cus + 1, 0, kEncPrime, kEncComplex, cus};  // of N = 8192
  if (log_n == 13 && n <= 2 * cus && primes > (beside ? 1 : 2)) return counted;
  if (n <= 2 * cus || (log_n < 13 && n <= 4 * cus)) return prime;
  if (beside) {
    if (log_n == 13 && n <= (primes < 8 ? 6 : 5) * cus) return by_n;
    if (log_n == 13) {
      const uint32_t share = n <= 64 * cus ? (primes < 3 ? 3 : 2) : (primes < 3 ? 5 : 3);
      return MissRoute{0, share, kEncComplex, kEncComplex, cus};
    }
    if (log_n == 12) return MissRoute{0, 1, kEncPrime, kEncComplex, 0};
    return MissRoute{0, 2, kEncPrime, kEncPrime, 2 * cus};
  }
  if (log_n == 13) return counted;
  const uint32_t from = (log_n == 11 ? 16 : primes < 8 ? 12 : 6) * (uint32_t)cus;
  if (n < from || (log_n == 11 && primes < 8)) return prime;
  return MissRoute{from, 0, kEncPrime, kEncComplex, 0};
}

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
