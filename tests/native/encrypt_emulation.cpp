// Host emulation of a row of the complex-transform encryption, down to its last step: the transforms
// of the emulation beside this file, then the kernel's own encrypt_residue.  Also the quotient of
// fft_combine by itself.
#include "fft_emulation.cpp"

namespace {

// One row: v wide + e + rint(fv cos) + rint(fb cos) mod q, as the kernel forms it; e given with its
// offset B, fv and fb only for polynomial 0.
template <int LOGN, int RC, int POLY>
void row(const double *v, const uint64_t *wide, uint64_t q, const uint32_t *e, int B, double fv, double fb, uint64_t *out) {
  using F = Fft<LOGN>;
  constexpr double unit = Split<RC>::unit;
  constexpr int N = 1 << LOGN, M = F::M;
  const Tables tb(LOGN);
  const double qd = (double)q, qinv = 1.0 / qd;
  std::vector<double> lo(N), hi(N);
  for (int j = 0; j < N; j++) {
    const double w = (double)wide[j], c = w > 0.5 * qd ? w - qd : w;
    hi[j] = __builtin_rint(c * (1.0 / unit));
    lo[j] = __builtin_fma(-hi[j], unit, c);
  }
  auto V = load<LOGN>(v);
  forward<LOGN>(V, tb);
  std::vector<Regs> X[2];
  for (int i = 0; i < 2; i++) {
    X[i] = load<LOGN>(i ? hi.data() : lo.data());
    forward<LOGN>(X[i], tb);
    for (int t = 0; t < F::T; t++)
      for (int r = 0; r < 16; r++) {
        double &xr = X[i][t].x[0][r], &xi = X[i][t].x[1][r];
        const double kr = xr * (1.0 / M), ki = xi * (1.0 / M), vr = V[t].x[0][r], vi = V[t].x[1][r];
        xr = __builtin_fma(vr, kr, -(vi * ki));
        xi = __builtin_fma(vr, ki, vi * kr);
      }
    inverse<LOGN>(X[i], tb);
  }
  const std::vector<double> cosj = host::cos_table(LOGN);
  for (int t = 0; t < F::T; t++) {
    const unsigned p = fft_place<LOGN>(t);
    for (int r = 0; r < 16; r++) {
      const Cplx tw = POLY == 0 ? Cplx{cosj[p + F::T * r], cosj[p + F::T * r + M]} : fft_twist(Cplx{cosj[p], cosj[p + M]}, r);
      for (int im = 0; im < 2; im++) {
        const double tr = im ? tw.im : tw.re, ti = im ? tw.re : -tw.im;
        const unsigned j = p + F::T * r + M * im;
        double add = (double)e[j];
        if (POLY == 0) add += __builtin_rint(fv * tr) + __builtin_rint(fb * tr);
        const double l = __builtin_fma(tr, X[0][t].x[0][r], __builtin_fma(ti, X[0][t].x[1][r], add));
        const double h = __builtin_rint(__builtin_fma(tr, X[1][t].x[0][r], ti * X[1][t].x[1][r]));
        out[j] = encrypt_residue<LOGN, RC, POLY>(h, l, qd, qinv, qinv * unit, (double)B);
      }
    }
  }
}

template <int LOGN>
void row_of(const double *v, const uint64_t *wide, uint64_t q, int rc, int poly, const uint32_t *e, int B, double fv,
            double fb, uint64_t *out) {
  if (rc)
    poly ? row<LOGN, 1, 1>(v, wide, q, e, B, fv, fb, out) : row<LOGN, 1, 0>(v, wide, q, e, B, fv, fb, out);
  else
    poly ? row<LOGN, 0, 1>(v, wide, q, e, B, fv, fb, out) : row<LOGN, 0, 0>(v, wide, q, e, B, fv, fb, out);
}

}  // namespace

extern "C" {

int emu_encrypt_row(int log_n, const double *v, const uint64_t *wide, uint64_t q, int rc, int poly, const uint32_t *e, int B,
                    double fv, double fb, uint64_t *out) {
  switch (log_n) {
    case 11: row_of<11>(v, wide, q, rc, poly, e, B, fv, fb, out); return 0;
    case 12: row_of<12>(v, wide, q, rc, poly, e, B, fv, fb, out); return 0;
    case 13: row_of<13>(v, wide, q, rc, poly, e, B, fv, fb, out); return 0;
    case 14: row_of<14>(v, wide, q, rc, poly, e, B, fv, fb, out); return 0;
    default: return -1;
  }
}

// out[i] = fft_combine(hi[i], w[i]) and wrap_center of it.
void emu_combine(const double *hi, const double *w, int n, int rc, uint64_t q, double *out, double *centered) {
  const double unit = rc ? Split<1>::unit : Split<0>::unit, qd = (double)q, qinv = 1.0 / qd;
  for (int i = 0; i < n; i++) {
    out[i] = fft_combine(hi[i], w[i], unit, qd, qinv, qinv * unit);
    centered[i] = wrap_center(out[i], qd);
  }
}
}
