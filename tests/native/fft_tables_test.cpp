// Host test of the complex transforms' factors (host::fft_tables): each part within 0.51 2^-53 of the
// extended-precision function of its angle, so that a factor is off by at most the 0.8 2^-53 that
// the proof of exactness allows.  Prints "OK".
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "../../paper_2409_03568_amd/csrc/host_math.hpp"

static int bad = 0;

// re, im against exp(i pi n / 2M)
static void check(const std::vector<double> &t, int64_t at, int64_t n, int64_t M, const char *what) {
  n %= 4 * M;
  const long double a = acosl(-1.0L) * (long double)(n > 2 * M ? n - 4 * M : n) / (long double)(2 * M);
  const long double want[2] = {cosl(a), sinl(a)};
  for (int k = 0; k < 2; k++) {
    const double got = t[(size_t)(2 * at + k)];
    if (!(fabsl((long double)got - want[k]) <= ldexpl(0.51L, -53))) {
      printf("%s %lld part %d: %.17g against %.17Lg\n", what, (long long)n, k, got, want[k]);
      bad++;
    }
  }
}

int main() {
  for (int log_n = 11; log_n <= 14; log_n++) {
    std::vector<double> fwd, inv;
    ckks::host::fft_tables(log_n, fwd, inv);
    const int64_t M = (int64_t)1 << (log_n - 1), T = M / 16;
    const int lm = log_n - 1;
    // inverse: exp(-i pi p / 2^bit) at the thread's place for bit lm - 1, and the middle pass's
    for (int64_t p = 0; p < T; p++) check(inv, p, 8 * M - (p << (lm + 1 - (lm - 1))), M, "inverse");
    for (int64_t p = 0; p < 16; p++) check(inv, T + 256 + p, 8 * M - (p << (lm + 1 - 7)), M, "inverse middle");
    // forward, low pass: node factors of element bit 0
    int64_t at = 4 + (M >> 8);
    for (int64_t h = 0; h < T; h++) {
      int64_t n = 1;
      for (int i = 0; 1 + i < lm; i++)
        if (((h << 4) >> (1 + i)) & 1) n += (int64_t)1 << (lm - i);
      check(fwd, at + h, n, M, "forward");
    }
  }
  if (!bad) printf("OK\n");
  return bad != 0;
}
