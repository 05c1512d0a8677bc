// Host emulation of the library's complex transforms (fft.hpp) for CPU tests: the level
// functions run for one emulated workgroup, thread by thread between the trades of lane bits
// and the LDS exchanges.
#include <math.h>
#include <stdint.h>

#include <algorithm>
#include <vector>

#include "../../paper_2409_03568_amd/csrc/fft.hpp"
#include "../../paper_2409_03568_amd/csrc/host_math.hpp"
#include "../../paper_2409_03568_amd/csrc/philox.hpp"

using namespace ckks;

namespace {

struct Regs {  // the registers of one thread: real and imaginary parts
  double x[2][16];
};

int g_layout_ok = 1;

struct Tables {
  std::vector<Cplx> fwd, inv;
  explicit Tables(int log_n) {
    std::vector<double> t[2];
    host::fft_tables(log_n, t[0], t[1]);
    for (int k = 0; k < 2; k++)
      for (size_t i = 0; i < t[k].size(); i += 2) (k ? inv : fwd).push_back(Cplx{t[k][i], t[k][i + 1]});
  }
};

// Trade of register bit 3 with lane bit 5: the upper half of register r with the lower half of
// register r + 8.
void trade(std::vector<Regs> &X) {
  for (size_t t = 0; t < X.size(); t++)
    if (!(t & 32))
      for (int c = 0; c < 2; c++)
        for (int r = 0; r < 8; r++) std::swap(X[t | 32].x[c][r], X[t].x[c][r + 8]);
}

// Which elements a layout holds: every one once; quarter-waves on 16 different 8-byte banks.
template <int LOGN, int PASS, bool DOWN>
void check_layout() {
  using F = Fft<LOGN>;
  std::vector<int> hit(F::M, 0);
  for (int r = 0; r < 16; r++)
    for (int t0 = 0; t0 < F::T; t0 += 16) {
      unsigned banks = 0;
      for (int t = t0; t < t0 + 16; t++) {
        const unsigned a = fft_thread<LOGN, PASS, DOWN>(t), b = fft_reg<LOGN, PASS, DOWN>(r);
        if (a & b) g_layout_ok = 0;
        if ((fft_slot(a) ^ fft_slot(b)) != fft_slot(a | b)) g_layout_ok = 0;
        hit[a | b]++;
        banks |= 1u << (fft_slot(a | b) & 15u);
      }
      if (banks != 0xffffu) g_layout_ok = 0;
    }
  for (int h : hit) g_layout_ok = g_layout_ok && h == 1;
}

template <int LOGN, int FROM, bool FD, int TO, bool TD>
void exchange(std::vector<Regs> &X) {
  using F = Fft<LOGN>;
  check_layout<LOGN, FROM, FD>();
  check_layout<LOGN, TO, TD>();
  std::vector<double> space(2 * F::M + 16);
  double *lds = (double *)(((uintptr_t)space.data() + 127) & ~(uintptr_t)127);
  for (int t = 0; t < F::T; t++) fft_store<LOGN, FROM, FD>(fft_base<LOGN, FROM, FD>(lds, t), X[t].x);
  if (F::same_wave_sets(FROM, TO))  // no workgroup barrier: every wave reads the slots it wrote
    for (int w = 0; w * 64 < F::T; w++) {
      std::vector<unsigned> wr, rd;
      for (int t = w * 64; t < w * 64 + 64; t++)
        for (int r = 0; r < 16; r++) {
          wr.push_back(fft_slot(fft_thread<LOGN, FROM, FD>(t) | fft_reg<LOGN, FROM, FD>(r)));
          rd.push_back(fft_slot(fft_thread<LOGN, TO, TD>(t) | fft_reg<LOGN, TO, TD>(r)));
        }
      std::sort(wr.begin(), wr.end());
      std::sort(rd.begin(), rd.end());
      g_layout_ok = g_layout_ok && wr == rd;
    }
  for (int t = 0; t < F::T; t++) fft_load<LOGN, TO, TD>(fft_base<LOGN, TO, TD>(lds, t), X[t].x);
}

template <int LOGN, int PASS, bool FWD>
void pass(std::vector<Regs> &X, const Tables &tb) {
  constexpr bool traded = PASS == kTop && Fft<LOGN>::trade;
  auto seg = [&](auto f) {
    for (int t = 0; t < Fft<LOGN>::T; t++)
      f(X[t].x, FWD ? fft_tw_fwd<LOGN, PASS>(t, tb.fwd.data()) : fft_tw_inv<LOGN, PASS>(t, tb.inv.data()));
  };
  if (FWD) {
    seg([](auto &x, const FftTw &f) { fft_fwd_levels<LOGN, PASS, 0>(x, f); });
    if (traded) {
      trade(X);
      seg([](auto &x, const FftTw &f) { fft_fwd_levels<LOGN, PASS, 1>(x, f); });
    }
  } else {
    if (traded) {
      seg([](auto &x, const FftTw &f) { fft_inv_levels<LOGN, PASS, 1>(x, f); });
      trade(X);
    }
    seg([](auto &x, const FftTw &f) { fft_inv_levels<LOGN, PASS, 0>(x, f); });
  }
}

template <int LOGN>
void forward(std::vector<Regs> &X, const Tables &tb) {
  pass<LOGN, kTop, true>(X, tb);
  exchange<LOGN, kTop, true, kMid, false>(X);
  pass<LOGN, kMid, true>(X, tb);
  exchange<LOGN, kMid, true, kLow, false>(X);
  pass<LOGN, kLow, true>(X, tb);
}
template <int LOGN>
void inverse(std::vector<Regs> &X, const Tables &tb) {
  pass<LOGN, kLow, false>(X, tb);
  exchange<LOGN, kLow, false, kMid, true>(X);
  pass<LOGN, kMid, false>(X, tb);
  exchange<LOGN, kMid, false, kTop, true>(X);
  pass<LOGN, kTop, false>(X, tb);
}

template <int LOGN>
std::vector<Regs> load(const double *a) {
  using F = Fft<LOGN>;
  std::vector<Regs> X(F::T);
  std::vector<int> hit(2 * F::M, 0);
  for (int t = 0; t < F::T; t++)
    for (int r = 0; r < 32; r++) {
      const unsigned j = fft_place<LOGN>(t) + F::T * r;
      if ((fft_thread<LOGN, kTop, false>(t) | fft_reg<LOGN, kTop, false>(r & 15)) != j % F::M) g_layout_ok = 0;
      X[t].x[r >> 4][r & 15] = a[j];
      hit[j]++;
    }
  for (int h : hit) g_layout_ok = g_layout_ok && h == 1;
  return X;
}

// c = small * wide mod q in Z[X]/(X^N + 1), small in {-1, 0, 1}, wide canonical (centered
// before the split when `center`): the steps of the kernels.  *off: the largest distance of a
// piece's coefficient from an integer.
template <int LOGN, int RC>
int product(const double *small, const uint64_t *wide, int center, uint64_t q, uint64_t *c, double *off) {
  using F = Fft<LOGN>;
  constexpr double unit = Split<RC>::unit;
  constexpr int N = 1 << LOGN, M = F::M;
  const Tables tb(LOGN);
  const double qd = (double)q, qinv = 1.0 / qd;
  std::vector<double> lo(N), hi(N);
  for (int j = 0; j < N; j++) {
    double v = (double)wide[j];
    if (center && v > 0.5 * qd) v -= qd;
    hi[j] = __builtin_rint(v * (1.0 / unit));
    lo[j] = __builtin_fma(-hi[j], unit, v);
  }
  auto S = load<LOGN>(small), A = load<LOGN>(lo.data()), B = load<LOGN>(hi.data());
  forward<LOGN>(S, tb);
  *off = 0;
  for (auto *X : {&A, &B}) {
    forward<LOGN>(*X, tb);
    for (int t = 0; t < F::T; t++)
      for (int r = 0; r < 16; r++) {
        double &xr = (*X)[t].x[0][r], &xi = (*X)[t].x[1][r];
        const double kr = S[t].x[0][r] * (1.0 / M), ki = S[t].x[1][r] * (1.0 / M);
        const double re = __builtin_fma(xr, kr, -(xi * ki)), im = __builtin_fma(xr, ki, xi * kr);
        xr = re;
        xi = im;
      }
    inverse<LOGN>(*X, tb);
    const std::vector<double> cosj = host::cos_table(LOGN);
    for (int t = 0; t < F::T; t++)
      for (int r = 0; r < 16; r++) {
        const unsigned p = fft_place<LOGN>(t);
        const Cplx w = fft_twist(Cplx{cosj[p], cosj[p + M]}, r);
        double &xr = (*X)[t].x[0][r], &xi = (*X)[t].x[1][r];
        const double re = __builtin_fma(w.re, xr, -(w.im * xi)), im = __builtin_fma(w.re, xi, w.im * xr);
        *off = std::max({*off, fabs(re - __builtin_rint(re)), fabs(im - __builtin_rint(im))});
        xr = __builtin_rint(re);
        xi = __builtin_rint(im);
      }
  }
  for (int t = 0; t < F::T; t++)
    for (int r = 0; r < 32; r++) {
      const double l = A[t].x[r >> 4][r & 15], h = B[t].x[r >> 4][r & 15];
      const double v = fft_combine(h, l, unit, qd, qinv, qinv * unit);
      if (fabs(v) > 0.5 * qd + 1) return -3;
      c[fft_place<LOGN>(t) + F::T * r] = (uint64_t)wrap_positive(v, qd);
      const double z = wrap_center(v, qd);
      if (!(z > -0.5 * qd && z <= 0.5 * qd) || wrap_positive(z, qd) != wrap_positive(v, qd)) return -4;
    }
  return 0;
}

}  // namespace

extern "C" {

// Words whose guided search and plain search differ: around every threshold, at the ends of every
// range of the guide, and `n` given ones.
int emu_guide_mismatches(double sigma, int B, const uint64_t *words, int n) {
  const std::vector<uint64_t> cdt = ckks::host::cdt_table(sigma, B, ckks::kCdtSlots);
  const std::vector<uint8_t> guide = ckks::host::cdt_guide(cdt, B, ckks::kGuideBits, ckks::kGuideMore);
  std::vector<uint64_t> w(words, words + n);
  for (int j = 0; j < 2 * B; j++)
    for (int d = -2; d <= 2; d++) w.push_back(cdt[j] + (uint64_t)(int64_t)d);
  for (uint64_t i = 0; i < (1u << ckks::kGuideBits); i++)
    for (int d = -1; d <= 1; d++) w.push_back((i << (64 - ckks::kGuideBits)) + (uint64_t)(int64_t)d);
  int bad = 0;
  for (uint64_t x : w)
    bad += ckks::gauss_of(x, cdt.data(), B) + B != (int)ckks::gauss_guided(x, cdt.data(), guide.data(), B);
  return bad;
}

int emu_fft_product(const double *small, const uint64_t *wide, int center, int log_n, uint64_t q, int rc, uint64_t *c,
                    double *off) {
  g_layout_ok = 1;
  switch (log_n) {
    case 11: return rc ? product<11, 1>(small, wide, center, q, c, off) : product<11, 0>(small, wide, center, q, c, off);
    case 12: return rc ? product<12, 1>(small, wide, center, q, c, off) : product<12, 0>(small, wide, center, q, c, off);
    case 13: return rc ? product<13, 1>(small, wide, center, q, c, off) : product<13, 0>(small, wide, center, q, c, off);
    case 14: return rc ? product<14, 1>(small, wide, center, q, c, off) : product<14, 0>(small, wide, center, q, c, off);
    default: return -1;
  }
}

int emu_fft_layout_ok(void) { return g_layout_ok; }
}
