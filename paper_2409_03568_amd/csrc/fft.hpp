// Negacyclic products with a small factor through complex FP64 transforms.
//
// Encryption multiplies the ternary polynomial v by the public key and decryption
// multiplies c1 by the ternary secret s (Sec. 2.2.2).  The integer coefficients of such a
// product are below N q, about 2^63, too wide for a double, but when the wide factor is
// split at 2^h into two pieces of about 25 bits each, both partial products fit with room to
// spare and are recovered exactly by rounding: an integer transform of the prime field (8
// operations per butterfly, one transform of v per prime) is replaced by a complex one (6
// fused multiply-adds per butterfly on half as many points, one transform of v for all
// primes).  Per ciphertext of N = 8192 and 4 primes: 17 complex transforms, 2.7 M FP64
// operations, instead of 12 prime-field ones, 5.1 M.
//
// Transform.  X^N + 1 = (X^M - i)(X^M + i) over C with M = N/2, so a real polynomial a is
// determined by a mod X^M - i, the M complex values z_j = a_j + i a_{j+M}.  The forward
// transform is the Cooley-Tukey network of X^M - i (each node X^2n - r^2 splits into X^n - r
// and X^n + r; no separate twist), output in bit-reversed order.  The inverse is the
// decimation-in-time network on that order (factor before the butterfly, so it fuses into
// multiply-adds as well) followed by the twist exp(-i pi j / 2M); 1/M is folded into the key
// tables.  Nodes that differ in their last bit differ by the factor i, so half the factors
// need no product.
//
// Work split: T = M/16 threads per ciphertext, 16 complex values each, so a pass does four
// levels between registers: element bits 0..3 (low pass), 4..7 (middle) and the rest (top, 2
// to 5 levels; the fifth, at N = 2^14, after a register bit has traded places with lane bit 5).
// Two exchanges per transform, the one between low and middle inside a wave.  A CU's LDS takes
// stores at 64 bytes per cycle, so with 8 values per thread (three levels per pass) the three
// exchanges of a transform, not its arithmetic, bounded it; passes of four levels on 8 values,
// the fourth after a trade with a lane bit, spent a sixth of their issue slots on the trades.
//
// Exactness.  Let u = 2^-53.  A butterfly o = fma(Wr, Y, fma(Wi, iY, X)), e = 2X - o is off by
// at most 3u (|X| + |Y|) plus |Y| times the error of W: 0.8u as loaded, 3u, 7.5u and 16.5u
// after one to three squarings, 2.8u more after a constant.  Averaged over a pass of four levels
// that is below 12u (|X| + |Y|) per level.  So the forward transforms of a and b lose at most
// 12u log M of their 2-norm each, which moves a coefficient of the product by at most 24u log M ||a||_2 ||b||_2;
// the errors of the inverse add up along the way to one coefficient to at most 12u log M times
// the mean of |a_hat b_hat|, which is at most ||a||_2 ||b||_2 (Cauchy-Schwarz); the pointwise
// product and the twist add 9u of it.  With ||a||_2 <= sqrt(N) (a ternary) and ||b||_2 <= 2^25
// sqrt(N) (a piece) every coefficient is within 12u (3 log M + 1) 2^25 N of its integer: 2^-6.2
// at N = 8192, 2^-5.1 at N = 2^14, for any input, against the 1/2 that rounding tolerates.
// Measured by the CPU tests: 2^-18 on random inputs, 2^-12 on the most extreme ones.
#pragma once
#include "ntt.hpp"

namespace ckks {

struct alignas(16) Cplx {
  double re, im;
};
typedef double f64x2 __attribute__((ext_vector_type(2)));

// Value `lane` of a uniform row of complex values (see row_at).
__device__ __forceinline__ Cplx ld_row(const Cplx *row, unsigned lane) {
  const f64x2 v = *row_at(reinterpret_cast<const f64x2 *>(row), lane);
  return Cplx{v.x, v.y};
}
CKKS_HD Cplx ld_cplx(const Cplx *__restrict__ base, unsigned idx) {
  return *reinterpret_cast<const Cplx *>(reinterpret_cast<const char *>(base) + (idx << 4));
}

// Bits of the low piece of a residue: pieces of at most 25 bits for q < 2^50 (class 1), of
// 20 for q < 2^40 (class 0).
template <int RC>
struct Split {
  static constexpr int bits = RC ? 25 : 20;
  static constexpr double unit = RC ? 33554432.0 : 1048576.0;  // 2^bits
};

// ---------------------------------------------------------------------------
// layouts
// ---------------------------------------------------------------------------
enum FftPass : int { kTop = 0, kMid = 1, kLow = 2 };

// Register r of thread tid holds one element per pass; the register bits are bits base ..
// base + 3 of it (top pass: the highest four).  In the top pass thread tid thus holds
// coefficients place + T r and place + T r + M, r < 16, the order coefficients are loaded and
// stored in; place is tid, except at N = 2^14, whose top pass trades register bit 3 with lane
// bit 5 for its fifth level (`down`: the layout on the middle pass's side of the trade).
template <int LOGN>
struct Fft {
  static constexpr int LM = LOGN - 1, M = 1 << LM, RB = 4, C = 16, T = M / C;
  static constexpr int top_levels = LM - 8;  // 2..5
  static constexpr bool trade = top_levels > RB;
  static constexpr int levels(int pass) { return pass == kTop ? top_levels : 4; }
  // element bit of register bit 0
  static constexpr int base(int pass) { return pass == kTop ? LM - RB : pass == kMid ? 4 : 0; }
  // exchanges inside a wave: low and middle pass keep the wave index at element bits 10 and up;
  // with one wave per workgroup all do
  static constexpr bool same_wave_sets(int a, int b) { return T <= 64 || (a != kTop && b != kTop); }
};

// Element bits of register r, of thread tid, in a layout; the two parts are disjoint.
template <int LOGN, int PASS, bool DOWN>
CKKS_HD constexpr unsigned fft_reg(unsigned r) {
  using F = Fft<LOGN>;
  if (PASS == kTop && F::trade && DOWN) return ((r & 7u) << 9) | ((r >> 3) << 8);
  return r << F::base(PASS);
}
template <int LOGN, int PASS, bool DOWN>
CKKS_HD unsigned fft_thread(unsigned tid) {
  using F = Fft<LOGN>;
  if constexpr (PASS == kLow) return tid << 4;
  if constexpr (PASS == kMid) return (tid & 15u) | ((tid >> 4) << 8);
  if constexpr (!F::trade) return tid;
  return (tid & 31u) | ((tid >> 6) << 5) | (((tid >> 5) & 1u) << (DOWN ? 12 : 8));
}

// The thread's place in the coefficient order.
template <int LOGN>
CKKS_HD unsigned fft_place(unsigned tid) { return fft_thread<LOGN, kTop, false>(tid); }

// LDS slot of element e: an XOR of the low four bits with the next four.  The 16 lanes of a
// quarter-wave differ in element bits 0..3 (top and middle pass) or 4..7 (low pass), which the
// slot maps one to one onto the 16 8-byte banks; it is linear over XOR, so a register adds a
// constant to a per-thread base after an XOR of four bits.
CKKS_HD constexpr unsigned fft_slot(unsigned e) { return e ^ ((e >> 4) & 15u); }

// A thread's base address in the exchange space for a layout, and its access to register r of a
// complex array from it: real parts at the slots, imaginary parts M further on (the same
// address register, another immediate offset).  The space is aligned to 128 bytes, so the XOR
// of a register's low slot bits can be taken on the address itself.
#if defined(__HIP_DEVICE_COMPILE__)
typedef uint32_t LdsAddr;
template <int LOGN, int PASS, bool DOWN>
CKKS_HD LdsAddr fft_base(double *lds, int tid) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds +
         (fft_slot(fft_thread<LOGN, PASS, DOWN>((unsigned)tid)) << 3);
}
CKKS_HD __attribute__((address_space(3))) double *lds_at(LdsAddr base, unsigned flip, unsigned offset) {
  return (__attribute__((address_space(3))) double *)(uintptr_t)((base ^ flip) + offset);
}
#else
typedef uintptr_t LdsAddr;
template <int LOGN, int PASS, bool DOWN>
CKKS_HD LdsAddr fft_base(double *lds, int tid) {
  return (uintptr_t)lds + (fft_slot(fft_thread<LOGN, PASS, DOWN>((unsigned)tid)) << 3);
}
CKKS_HD double *lds_at(LdsAddr base, unsigned flip, unsigned offset) { return (double *)((base ^ flip) + offset); }
#endif
template <int LOGN, int PASS, bool DOWN>
CKKS_HD void fft_store(LdsAddr base, const double (&x)[2][16]) {
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const unsigned pr = fft_slot(fft_reg<LOGN, PASS, DOWN>(r)), flip = (pr & 15u) << 3, at = (pr & ~15u) << 3;
    *lds_at(base, flip, at) = x[0][r];
    *lds_at(base, flip, at + 8 * Fft<LOGN>::M) = x[1][r];
  }
}
template <int LOGN, int PASS, bool DOWN>
CKKS_HD void fft_load(LdsAddr base, double (&x)[2][16]) {
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const unsigned pr = fft_slot(fft_reg<LOGN, PASS, DOWN>(r)), flip = (pr & 15u) << 3, at = (pr & ~15u) << 3;
    x[0][r] = *lds_at(base, flip, at);
    x[1][r] = *lds_at(base, flip, at + 8 * Fft<LOGN>::M);
  }
}

// Trades register bit 3 with lane bit 5: the upper half of register r with the lower half of
// register r + 8.
__device__ __forceinline__ void fft_trade(double (&x)[2][16]) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int c = 0; c < 2; c++)
#pragma unroll
    for (int r = 0; r < 8; r++) {
      const uint64_t a = __builtin_bit_cast(uint64_t, x[c][r]), b = __builtin_bit_cast(uint64_t, x[c][r + 8]);
      const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)a, (uint32_t)b, false, false);
      const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(a >> 32), (uint32_t)(b >> 32), false, false);
      x[c][r] = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
      x[c][r + 8] = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
    }
#endif
}

// ---------------------------------------------------------------------------
// butterflies and factors
// ---------------------------------------------------------------------------
// (X, Y) -> (X + W Y, X - W Y) in six fused multiply-adds.
CKKS_HD void cx_butterfly(double &Xr, double &Xi, double &Yr, double &Yi, double Wr, double Wi) {
  const double or_ = __builtin_fma(Wr, Yr, __builtin_fma(-Wi, Yi, Xr));
  const double oi = __builtin_fma(Wr, Yi, __builtin_fma(Wi, Yr, Xi));
  Yr = __builtin_fma(2.0, Xr, -or_);
  Yi = __builtin_fma(2.0, Xi, -oi);
  Xr = or_;
  Xi = oi;
}
constexpr double kCosPi4 = 0.70710678118654752440, kCosPi8 = 0.92387953251128675613, kSinPi8 = 0.38268343236508977173;
CKKS_HD Cplx cx_mul(Cplx a, double re, double im) {
  return Cplx{__builtin_fma(a.re, re, -(a.im * im)), __builtin_fma(a.re, im, a.im * re)};
}
// a exp(+-i pi e / 8), e = 0..3
CKKS_HD Cplx cx_turn(Cplx a, int e, bool positive) {
  const double s = positive ? 1.0 : -1.0;
  if (e == 0) return a;
  if (e == 2) return Cplx{(a.re - s * a.im) * kCosPi4, (a.im + s * a.re) * kCosPi4};
  return e == 1 ? cx_mul(a, kCosPi8, s * kSinPi8) : cx_mul(a, kSinPi8, s * kCosPi8);
}
// square of a unit value
CKKS_HD Cplx cx_square(Cplx a) {
  const double t = a.im + a.im;
  return Cplx{__builtin_fma(-t, a.im, 1.0), t * a.re};
}

// One level of a transform on 16 values: butterflies along register bit K.  The factor is base
// times exp(+-i pi / 2), / 4 and / 8 for each set bit among up to three other register bits B1,
// B2, B3 (-1: none), + forward, - inverse.  UNIT: base is 1.
template <int K, int B1, int B2, int B3, bool FWD, bool UNIT = false>
CKKS_HD void fft_level(double (&x)[2][16], Cplx base) {
#pragma unroll
  for (int e = 0; e < 4; e++) {  // eighths of a half turn besides those of B1
    if ((B2 < 0 && e >= 2) || (B3 < 0 && (e & 1))) continue;
    const Cplx w = cx_turn(UNIT ? Cplx{1.0, 0.0} : base, e, FWD);
#pragma unroll
    for (int r = 0; r < 16; r++) {
      if (r & (1 << K)) continue;
      auto bit = [&](int k) { return k < 0 ? 0 : (r >> k) & 1; };
      if (2 * bit(B2) + bit(B3) != e) continue;
      double &Xr = x[0][r], &Xi = x[1][r], &Yr = x[0][r | (1 << K)], &Yi = x[1][r | (1 << K)];
      const bool turn = bit(B1) != 0;
      if (UNIT && e == 0) {  // factor 1 or +-i
        const double yr = turn ? (FWD ? -Yi : Yi) : Yr, yi = turn ? (FWD ? Yr : -Yr) : Yi;
        const double re = Xr - yr, im = Xi - yi;
        Xr += yr;
        Xi += yi;
        Yr = re;
        Yi = im;
      } else if (turn) {
        cx_butterfly(Xr, Xi, Yr, Yi, FWD ? -w.im : w.im, FWD ? w.re : -w.re);
      } else {
        cx_butterfly(Xr, Xi, Yr, Yi, w.re, w.im);
      }
    }
  }
  stage_fence();
}

// The loaded factors of a thread in one pass.  Forward, with h the element bits above the
// pass: w0 is the factor of the last level between registers, whose squares serve the levels
// before it.  Inverse, with off the element bits below: w0 belongs to the last level (the
// largest distance), its squares to the levels before it.  w1: the level on the other side of
// the trade at N = 2^14 (forward the last, inverse the first).
struct FftTw {
  Cplx w0, w1;
};

// Places of the factors in the tables (host_math.cpp fills them):
//   forward: top pass w0 at 0, w1 at 2 + lane bit 5; a lower pass from fwd_at: w0 at h;
//   inverse: top pass w0 at the thread's place, w1 from inv_top1; middle pass w0 from inv_mid.
template <int LOGN>
struct FftTables {
  using F = Fft<LOGN>;
  static constexpr unsigned fwd_at(int pass) { return pass == kMid ? 4 : 4 + (1u << (F::LM - 8)); }
  static constexpr unsigned inv_top1 = F::T, inv_mid = F::T + 256;
  static_assert(fwd_at(kLow) + F::T <= (unsigned)F::M && inv_mid + 16 <= (unsigned)F::M, "tables of M values");
};

template <int LOGN, int PASS>
CKKS_HD FftTw fft_tw_fwd(int tid_in, const Cplx *__restrict__ tw) {
  using B = FftTables<LOGN>;
  const unsigned tid = (unsigned)opaque(tid_in);
  FftTw f{};
  if constexpr (PASS == kTop) {
    f.w0 = ld_cplx(tw, 0);
    if constexpr (Fft<LOGN>::trade) f.w1 = ld_cplx(tw, 2 + ((tid >> 5) & 1u));
  } else {
    f.w0 = ld_cplx(tw, B::fwd_at(PASS) + (fft_thread<LOGN, PASS, false>(tid) >> (PASS == kMid ? 8 : 4)));
  }
  return f;
}

template <int LOGN, int PASS>
CKKS_HD FftTw fft_tw_inv(int tid_in, const Cplx *__restrict__ tw) {
  using B = FftTables<LOGN>;
  const unsigned tid = (unsigned)opaque(tid_in);
  FftTw f{};
  if constexpr (PASS == kTop) {
    const unsigned p = fft_place<LOGN>(tid);
    f.w0 = ld_cplx(tw, p);
    if constexpr (Fft<LOGN>::trade) f.w1 = ld_cplx(tw, B::inv_top1 + (p & 255u));
  } else if constexpr (PASS == kMid) {
    f.w0 = ld_cplx(tw, B::inv_mid + (tid & 15u));
  }
  return f;  // low pass: constants
}

// The levels of a pass between registers; of the traded level of the top pass at N = 2^14
// (SEG = 1: forward after, inverse before the trade).
template <int LOGN, int PASS, int SEG>
CKKS_HD void fft_fwd_levels(double (&x)[2][16], const FftTw &f) {
  constexpr int n = PASS == kTop && !Fft<LOGN>::trade ? Fft<LOGN>::top_levels : 4;
  if constexpr (SEG == 1) {
    // register bit 3 is element bit 8; bits 0..2 are 9..11, lane bit 5 (in w1) is 12
    fft_level<3, 0, 1, 2, true>(x, f.w1);
  } else {
    const Cplx s1 = cx_square(f.w0), s2 = cx_square(s1);
    if constexpr (n == 4) fft_level<3, -1, -1, -1, true>(x, cx_square(s2));
    if constexpr (n == 4) fft_level<2, 3, -1, -1, true>(x, s2);
    if constexpr (n == 4) fft_level<1, 2, 3, -1, true>(x, s1);
    if constexpr (n == 4) fft_level<0, 1, 2, 3, true>(x, f.w0);
    if constexpr (n == 3) fft_level<3, -1, -1, -1, true>(x, s2);
    if constexpr (n == 3) fft_level<2, 3, -1, -1, true>(x, s1);
    if constexpr (n == 3) fft_level<1, 2, 3, -1, true>(x, f.w0);
    if constexpr (n == 2) fft_level<3, -1, -1, -1, true>(x, s1);
    if constexpr (n == 2) fft_level<2, 3, -1, -1, true>(x, f.w0);
  }
}
template <int LOGN, int PASS, int SEG>
CKKS_HD void fft_inv_levels(double (&x)[2][16], const FftTw &f) {
  constexpr int n = PASS == kTop && !Fft<LOGN>::trade ? Fft<LOGN>::top_levels : 4;
  constexpr bool unit = PASS == kLow;
  if constexpr (SEG == 1) {
    fft_level<3, -1, -1, -1, false>(x, f.w1);
  } else {
    // (after the trade lane bit 5, element bit 8, belongs to the place, so to the bases)
    const Cplx s1 = cx_square(f.w0), s2 = cx_square(s1);
    if constexpr (n == 4) fft_level<0, -1, -1, -1, false, unit>(x, cx_square(s2));
    if constexpr (n == 4) fft_level<1, 0, -1, -1, false, unit>(x, s2);
    if constexpr (n == 3) fft_level<1, 0, -1, -1, false>(x, s2);
    if constexpr (n >= 3) fft_level<2, 1, 0, -1, false, unit>(x, s1);
    if constexpr (n == 2) fft_level<2, 1, 0, -1, false>(x, s1);
    fft_level<3, 2, 1, 0, false, unit>(x, f.w0);
  }
}

template <int LOGN, int PASS, bool FWD>
__device__ __forceinline__ void fft_pass(double (&x)[2][16], FftTw f) {
  // each array forms the squares and constants again (25 instructions of about 420): kept for
  // the next array they would cost up to 24 registers (17.7 against 17.0 ms per 65,536 plain
  // encryptions at N = 8192)
  if constexpr (FWD || PASS != kLow) {
    computed_here(f.w0.re);
    computed_here(f.w0.im);
  }
  constexpr bool traded = PASS == kTop && Fft<LOGN>::trade;
  if constexpr (FWD) {
    fft_fwd_levels<LOGN, PASS, 0>(x, f);
    if constexpr (traded) {
      fft_trade(x);
      fft_fwd_levels<LOGN, PASS, 1>(x, f);
    }
  } else {
    if constexpr (traded) {
      fft_inv_levels<LOGN, PASS, 1>(x, f);
      fft_trade(x);
    }
    fft_inv_levels<LOGN, PASS, 0>(x, f);
  }
}

// The twist exp(-i pi (p + T r) / 2M) of register r from that of register 0: exp(-i pi r / 32)
// times it.
CKKS_HD Cplx fft_twist(Cplx t0, int r) {
  constexpr double c[17] = {1.0, 0.99518472667219688624, 0.98078528040323044913, 0.95694033573220886494,
                            0.92387953251128675613, 0.88192126434835502971, 0.83146961230254523708,
                            0.77301045336273696081, 0.70710678118654752440, 0.63439328416364549822,
                            0.55557023301960222474, 0.47139673682599764856, 0.38268343236508977173,
                            0.29028467725446236764, 0.19509032201612826785, 0.09801714032956060199, 0.0};
  return r == 0 ? t0 : cx_mul(t0, c[r], -c[16 - r]);
}

// ---------------------------------------------------------------------------
// transforms of NA arrays by one workgroup, through one LDS space of N doubles
// ---------------------------------------------------------------------------
// Exchange of one array between the layouts of two passes, from and to: the thread's base
// addresses in them.  `lead`: other waves may still read the space, so the store waits for them.
template <int LOGN, int FROM, bool FROM_DOWN, int TO, bool TO_DOWN>
__device__ __forceinline__ void fft_exchange(double (&x)[2][16], LdsAddr from, LdsAddr to, bool lead) {
  constexpr bool kLocal = Fft<LOGN>::same_wave_sets(FROM, TO);
  if (kLocal && !lead)
    wave_sync();
  else
    __syncthreads();
  fft_store<LOGN, FROM, FROM_DOWN>(from, x);
  exchange_mid<kLocal>();
  fft_load<LOGN, TO, TO_DOWN>(to, x);
  stage_fence();
}

// The arrays take turns through each pass and its exchange, so that one array's butterflies
// cover the other's LDS traffic (a wave's LDS accesses are performed in order, so the arrays
// share one space).  Every thread of the workgroup must call these (barriers).

// Coefficient order (up layout of the top pass) to transform order (down layout of the low
// pass).
template <int LOGN, int NA>
__device__ __forceinline__ void fft_forward(double (&x)[NA][2][16], double *lds, int tid, const Cplx *__restrict__ tw) {
  const FftTw top = fft_tw_fwd<LOGN, kTop>(tid, tw), mid = fft_tw_fwd<LOGN, kMid>(tid, tw);
  {
    const int t = opaque(tid);
    const LdsAddr from = fft_base<LOGN, kTop, true>(lds, t), to = fft_base<LOGN, kMid, false>(lds, t);
#pragma unroll
    for (int a = 0; a < NA; a++) {
      fft_pass<LOGN, kTop, true>(x[a], top);
      fft_exchange<LOGN, kTop, true, kMid, false>(x[a], from, to, a == 0);
    }
  }
  const FftTw low = fft_tw_fwd<LOGN, kLow>(tid, tw);
  {
    const int t = opaque(tid);
    const LdsAddr from = fft_base<LOGN, kMid, true>(lds, t), to = fft_base<LOGN, kLow, false>(lds, t);
#pragma unroll
    for (int a = 0; a < NA; a++) {
      fft_pass<LOGN, kMid, true>(x[a], mid);
      fft_exchange<LOGN, kMid, true, kLow, false>(x[a], from, to, false);
    }
  }
#pragma unroll
  for (int a = 0; a < NA; a++) fft_pass<LOGN, kLow, true>(x[a], low);
}

// Transform order to coefficient order (times M, without the twist).  before_last() runs before
// the last pass: a place for the caller's loads, whose latency then hides behind it.
template <int LOGN, int NA, class FN>
__device__ __forceinline__ void fft_inverse(double (&x)[NA][2][16], double *lds, int tid, const Cplx *__restrict__ tw,
                                            FN &&before_last) {
  const FftTw low = fft_tw_inv<LOGN, kLow>(tid, tw), mid = fft_tw_inv<LOGN, kMid>(tid, tw);
  {
    const int t = opaque(tid);
    const LdsAddr from = fft_base<LOGN, kLow, false>(lds, t), to = fft_base<LOGN, kMid, true>(lds, t);
#pragma unroll
    for (int a = 0; a < NA; a++) {
      fft_pass<LOGN, kLow, false>(x[a], low);
      // another wave may still be reading the space in coefficient order (an earlier inverse)
      fft_exchange<LOGN, kLow, false, kMid, true>(x[a], from, to, a == 0);
    }
  }
  const FftTw top = fft_tw_inv<LOGN, kTop>(tid, tw);
  {
    const int t = opaque(tid);
    const LdsAddr from = fft_base<LOGN, kMid, false>(lds, t), to = fft_base<LOGN, kTop, true>(lds, t);
#pragma unroll
    for (int a = 0; a < NA; a++) {
      fft_pass<LOGN, kMid, false>(x[a], mid);
      fft_exchange<LOGN, kMid, false, kTop, true>(x[a], from, to, false);
    }
  }
  before_last();
  stage_fence();
#pragma unroll
  for (int a = 0; a < NA; a++) fft_pass<LOGN, kTop, false>(x[a], top);
}

// Congruent to hi 2^h + w mod q for integer-valued hi (|hi| 2^h < 2^66) and w (|w| < 2^51,
// w + the result below 2^53).  qinv_u = 2^h / q.  H - c q is an integer below 2^53, so the fused
// multiply-add forms it exactly.  The quotient, of magnitude up to N, is rounded from a value off by
// up to N 2^-51, so |result| <= q/2 + N q 2^-51 + 1: past q/2 by up to 2^12 at N = 8192 and 50 bits.
// (wrap_center and encrypt_residue take anything below 3q/2 and q.)
CKKS_HD double fft_combine(double hi, double w, double unit, double q, double qinv, double qinv_u) {
  const double c = __builtin_rint(__builtin_fma(hi, qinv_u, w * qinv));
  return __builtin_fma(-c, q, hi * unit) + w;
}

// Centered residue, in (-q/2, q/2], of r with |r| < 3q/2 (q odd).
CKKS_HD double wrap_center(double r, double q) {
  return __builtin_fabs(r) > 0.5 * q ? r - __builtin_copysign(q, r) : r;
}

// Canonical residue of r in (-q, q).
CKKS_HD double wrap_positive(double r, double q) { return r < 0.0 ? r + q : r; }

// Last step of a row of encryption: the canonical residue of hi 2^h + lo - b, hi the rounded high
// piece of v pk, lo the low one plus everything added to it and the errors' offset b, not rounded yet.
template <int LOGN, int RC, int POLY>
CKKS_HD uint64_t encrypt_residue(double hi, double lo, double q, double qinv, double qinv_u, double b) {
  constexpr double unit = Split<RC>::unit;
  double c;  // c0 or c1, plus b, in (-q, q)
  if constexpr (RC == 0 && LOGN <= 12) {
    // |v pk| <= N q/2 <= 2^51: the sum of the pieces is exact
    const double y = __builtin_fma(hi, unit, __builtin_rint(lo));
    c = __builtin_fma(-__builtin_rint(y * qinv), q, y);
  } else if constexpr (RC == 1 && POLY == 1) {
    // |low piece| <= N 2^24 + 2B < q/2 (q > 2^40): the high piece alone gives the quotient
    c = __builtin_fma(-__builtin_rint(hi * qinv_u), q, hi * unit) + lo;
  } else {
    c = fft_combine(hi, lo, unit, q, qinv, qinv_u);
  }
  // without b, wrapped to [0, q) and rounded by the addition of 2^52: before it the low piece
  // was off its integer by under 2^-5, and the sums of magnitudes up to 2^50 by under 2^-1.3
  return __builtin_bit_cast(uint64_t, c + (c < b - 0.5 ? (kTwo52 - b) + q : kTwo52 - b)) - kTwo52Bits;
}

}  // namespace ckks
