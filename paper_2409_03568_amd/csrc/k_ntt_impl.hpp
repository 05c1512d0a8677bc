// Transform-based kernels: key generation (prime-field NTT, ntt.hpp) and key preparation,
// fused per-pixel encryption and decryption (complex transforms, fft.hpp).  One workgroup
// handles one ciphertext at a time (all limbs), so the random polynomials v, e0, e1 are drawn,
// and v transformed, once per ciphertext and reused by every limb.
//
// Template parameters: LOGN (ring degree), RC (class of the primes' sizes, see ntt.hpp and
// Split) and, for the kernels on prime-field transforms, LOGR (values per thread, so
// N / 2^LOGR threads per workgroup).  Each ring degree is instantiated in its own translation
// units (k_ntt_<LOGN>_*.hip).
#pragma once
#include <algorithm>
#include <atomic>

#include "fft.hpp"
#include "internal.hpp"
#include "ntt.hpp"
#include "philox.hpp"
#include "routes.hpp"

namespace ckks {

template <int LOGN, int LOGR>
struct Shape : NttShape<LOGN, LOGR> {
  static constexpr int LAST = NttShape<LOGN, LOGR>::NPASS - 1;
  // dynamic LDS: the exchange space (N doubles with padding, see lds_pos), the Gaussian
  // table, and a reduction area
  static constexpr int SLOTS = LdsSlots<LOGN, LOGR>::value;
  static constexpr size_t lds_bytes = sizeof(double) * ((size_t)SLOTS + kCdtSlots + 64);
  // encryption: then a second exchange space where it fits (N <= 8192; the two inverse transforms
  // of a limb then run as one paired transform), and the packed samples of the current ciphertext
  // where they fit too (else in registers); k_encrypt_ntt adds the samplers' guide, but at N = 2048
  // goes without: four workgroups share a CU there, with the guide's LDS three, and its loads cost
  // small calls more than its search saves (100 pixels 41.3 against 40.9 us, 8,000 428 against 411)
  static constexpr size_t smp_bytes = sizeof(uint16_t) << LOGN;
  static constexpr bool kDual = lds_bytes + sizeof(double) * (size_t)SLOTS <= 160 * 1024;
  static constexpr size_t enc_smp_at = lds_bytes + (kDual ? sizeof(double) * (size_t)SLOTS : 0);
  static constexpr bool kSmpLds = enc_smp_at + smp_bytes <= 160 * 1024;
  static constexpr size_t enc_lds_bytes = enc_smp_at + (kSmpLds ? smp_bytes : 0);
  static constexpr int enc_guide = LOGN == 11 ? 0 : kGuideBits;
  static constexpr size_t enc_guided_lds_bytes = enc_lds_bytes + (enc_guide ? 1 << enc_guide : 0);
};

// Draw the packed samples of one polynomial triple into LDS: word j of dst holds
// coefficient j as (t1 + 1) | (g2 + B) << 2 | (g3 + B) << 9, where t1 is the ternary
// value of stream tag1 and g2, g3 the Gaussian values of streams tag2, tag3 (all at
// Philox index t; 0 <= g + B <= 2B <= 126; streams that are not used leave any value).  Each of
// `threads` threads draws whole Philox blocks; ends with a barrier.  GUIDED: with the guide of gauss_guided.
constexpr int kSmpShiftG2 = 2, kSmpShiftG3 = 9;

template <int LOGN, bool GUIDED>
__device__ __forceinline__ void draw_samples(uint16_t *dst, const uint64_t *cdt, int B, int tid, int threads,
                                             uint64_t k0, uint64_t k1, uint64_t t, uint32_t tag1, uint32_t tag2,
                                             uint32_t tag3, bool use2, bool use3, const uint8_t *guide) {
#pragma unroll 1
  for (uint32_t b = (uint32_t)tid; b < (1u << LOGN) / 4; b += (uint32_t)threads) {
    const Philox4 pv = philox4x64_10(t, tag1, b, 0, k0, k1);
    const Philox4 pa = use2 ? philox4x64_10(t, tag2, b, 0, k0, k1) : Philox4{};
    const Philox4 pb = use3 ? philox4x64_10(t, tag3, b, 0, k0, k1) : Philox4{};
    uint32_t w2[2];
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const uint32_t tv = (uint32_t)(ternary_of(pv.w[w]) + 1);
      uint32_t ga, gb;
      if constexpr (GUIDED) {
        ga = gauss_guided(pa.w[w], cdt, guide, B);
        gb = gauss_guided(pb.w[w], cdt, guide, B);
      } else {
        ga = (uint32_t)(gauss_of(pa.w[w], cdt, B) + B);
        gb = (uint32_t)(gauss_of(pb.w[w], cdt, B) + B);
      }
      const uint32_t word = tv | (ga << kSmpShiftG2) | (gb << kSmpShiftG3);
      w2[w >> 1] = (w & 1) ? (w2[w >> 1] | (word << 16)) : word;
    }
    reinterpret_cast<uint2 *>(dst)[b] = make_uint2(w2[0], w2[1]);
  }
  __syncthreads();
}

// The same, read back in the first-pass layout: smp[r] holds coefficient tid + T*r.
template <int LOGN, int LOGR>
__device__ __forceinline__ void draw_samples(uint32_t (&smp)[1 << LOGR], uint16_t *lds16, const uint64_t *cdt,
                                             int B, int tid, uint64_t k0, uint64_t k1, uint64_t t, uint32_t tag1,
                                             uint32_t tag2, uint32_t tag3) {
  using S = NttShape<LOGN, LOGR>;
  draw_samples<LOGN, false>(lds16, cdt, B, tid, S::T, k0, k1, t, tag1, tag2, tag3, true, true, nullptr);
#pragma unroll
  for (int r = 0; r < S::R; r++) smp[r] = lds16[tid + S::T * r];
}

__device__ __forceinline__ int smp_t(uint32_t s) { return (int)(s & 3u) - 1; }
__device__ __forceinline__ int smp_g(uint32_t s, int shift, int B) { return (int)((s >> shift) & 0x7fu) - B; }

// ---------------------------------------------------------------------------
// fused plain encryption: c0 = v pk0 + e0 + m, c1 = v pk1 + e1 per limb.  v is transformed
// once; each row (one polynomial of one limb) takes the two inverse transforms of its pieces
// (see fft.hpp).
// ---------------------------------------------------------------------------
// LDS of the complex-transform kernels: the exchange space of N doubles (it also holds the
// Gaussian table while samples are drawn, and the decoding's sums); encryption adds the packed
// samples of the current ciphertext (2 bytes per coefficient), which N = 2^14 keeps in
// registers.  At N = 8192 that is 80 KiB: two workgroups share a CU, and one's arithmetic covers
// the other's barriers and loads.
template <int LOGN>
struct FftLds {
  static constexpr size_t exchange = sizeof(double) << LOGN;
  static constexpr bool kSmp = LOGN <= 13;
  static constexpr size_t encrypt = exchange + (kSmp ? sizeof(uint16_t) << LOGN : 0);
};

// Where item i's pixel value and Philox index come from (compiled separately, so each
// variant keeps only the pointers it reads live):
//   kEncPixels:  items 0..n-1, value px[i], index first_index + i;
//   kEncList:    items list[0..*list_count), value px[item], index first_index + item;
//   kEncEntries: items 0..count-1 (count = *list_count if set, else n), value vals[i],
//                index ts[i].
// BRIGHT adds the image's brightness encoding to c0 (EncJob::seg_b).
enum EncMode : int { kEncPixels = 0, kEncList = 1, kEncEntries = 2 };

// One encryption: its ciphertext's place, Philox index, and the factors of the encodings of its
// value and brightness, rint(fv cos(pi j / N)) with fv = value 2^(1 - log N) scale, exact as the
// value times a power of two.
struct EncItem {
  uint64_t slot, t;
  double fv, fb;
};
template <int MODE>
__device__ __forceinline__ uint64_t enc_count(const EncJob &job) {
  if (MODE == kEncEntries && job.list_count) return *job.list_count;
  if (MODE != kEncList) return job.n;
  if (!gate_open(job.gate, job.list_count)) return 0;
  const uint64_t m = *job.list_count, left = m > job.list_first ? m - job.list_first : 0;
  return left < job.n ? left : job.n;
}
template <int MODE, bool BRIGHT>
__device__ __forceinline__ EncItem enc_item(const EncJob &job, uint64_t it, const LimbConsts &lc) {
  const uint64_t item = MODE == kEncList ? (uint64_t)job.list[job.list_first + it] : it;
  EncItem e;
  e.slot = MODE == kEncList && job.compact ? it : item;
  e.t = MODE == kEncEntries ? job.ts[item] : job.first_index + item;
  e.fv = (MODE == kEncEntries ? (double)job.vals[item] : (double)job.px[item]) * lc.enc_scale;
  e.fb = BRIGHT ? job.seg_b[segment_of(job.seg_end, job.n_seg, job.seg_base + item)] * job.bright_scale : 0.0;
  return e;
}

// The samples of one encryption: packed words of coefficients p + T r (p the thread's place),
// in LDS or in registers.
template <int LOGN>
struct Samples {
  const uint16_t *lds;
  uint32_t reg[FftLds<LOGN>::kSmp ? 1 : 32];
  __device__ __forceinline__ uint32_t at(int r, int p) const {
    if constexpr (FftLds<LOGN>::kSmp)
      return (uint32_t)lds[p + Fft<LOGN>::T * r];
    else
      return reg[r];
  }
};

// Draws the samples of encryption t (the Gaussian ones of e0 and e1 if asked for) with the
// `threads` threads of the workgroup.  The Gaussian tables are staged in the exchange space, which
// another wave may still be using for an earlier item.
template <int LOGN>
__device__ __forceinline__ void draw_item(Samples<LOGN> &smp, double *lds, int B, uint64_t k0, uint64_t k1, uint64_t t,
                                          int threads, bool e0, bool e1, const DevTables &dt) {
  using F = Fft<LOGN>;
  const int tid = opaque(threadIdx.x);
  constexpr int kTable = kCdtSlots + (1 << kGuideBits) / (int)sizeof(uint64_t);  // thresholds and guide
  uint64_t *cdt = reinterpret_cast<uint64_t *>(lds);
  uint16_t *words = FftLds<LOGN>::kSmp ? reinterpret_cast<uint16_t *>(lds + 2 * F::M)
                                       : reinterpret_cast<uint16_t *>(cdt + kTable);
  __syncthreads();
  for (int i = tid; i < kTable / 2; i += threads)
    reinterpret_cast<u64x2 *>(cdt)[i] = reinterpret_cast<const u64x2 *>(dt.cdt)[i];
  __syncthreads();
  draw_samples<LOGN, true>(words, cdt, B, tid, threads, k0, k1, t, kTagV, kTagE0, kTagE1, e0, e1,
                           reinterpret_cast<const uint8_t *>(cdt + kCdtSlots));
  smp.lds = words;
  if constexpr (!FftLds<LOGN>::kSmp) {
    const int p = (int)fft_place<LOGN>((unsigned)tid);
#pragma unroll
    for (int r = 0; r < 32; r++) smp.reg[r] = words[p + F::T * r];
  }
}

// v_hat of the current item, in transform order.
template <int LOGN>
__device__ __forceinline__ void encrypt_forward(double (&v)[1][2][16], double *lds, const Samples<LOGN> &smp,
                                                const DevTables &dt) {
  const int tid = opaque(threadIdx.x), p = (int)fft_place<LOGN>((unsigned)tid);
#pragma unroll
  for (int r = 0; r < 32; r++) v[0][r >> 4][r & 15] = (double)smp_t(smp.at(r, p));
  fft_forward<LOGN, 1>(v, lds, tid, dt.fft_fwd);
#pragma unroll
  for (int r = 0; r < 32; r++) computed_here(v[0][r >> 4][r & 15]);
}

// A quarter of a row's key values: both pieces of values 4 part .. 4 part + 3.
struct KeyPart {
  Cplx k[4][2];
};
template <int LOGN>
__device__ __forceinline__ const Cplx *key_row(int poly, int l, int L, const DevTables &dt) {
  return dt.pk_fft + ((size_t)poly * L + l) * 2 * Fft<LOGN>::M;
}
template <int LOGN>
__device__ __forceinline__ KeyPart load_part(const Cplx *key, int part) {
  using F = Fft<LOGN>;
  const unsigned tid = (unsigned)opaque(threadIdx.x);
  KeyPart o;
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int i = 0; i < 2; i++) o.k[r][i] = ld_row(key + i * F::M + (4 * part + r) * F::T, tid);
  return o;
}
__device__ __forceinline__ void row_product(double (&x)[2][2][16], const double (&v)[1][2][16], const KeyPart &o, int part) {
#pragma unroll
  for (int r = 0; r < 4; r++)
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const int at = 4 * part + r;
      const double vr = v[0][0][at], vi = v[0][1][at];
      x[i][0][at] = __builtin_fma(vr, o.k[r][i].re, -(vi * o.k[r][i].im));
      x[i][1][at] = __builtin_fma(vr, o.k[r][i].im, vi * o.k[r][i].re);
      computed_here(x[i][0][at]);
      computed_here(x[i][1][at]);
    }
  stage_fence();
}

// Half of a row's results: coefficients p + T r and p + T r + M of values r = 8 h .. 8 h + 7.
struct RowHalf {
  uint64_t w[2][8];
};
template <int LOGN>
__device__ __forceinline__ void store_half(uint64_t *row, const RowHalf &res, int h) {
  using F = Fft<LOGN>;
  const unsigned p = fft_place<LOGN>((unsigned)opaque(threadIdx.x));
#pragma unroll
  for (int im = 0; im < 2; im++)
#pragma unroll
    for (int r = 0; r < 8; r++)
      __builtin_nontemporal_store(res.w[im][r], row_at(row + F::T * (8 * h + r) + F::M * im, p));
  stage_fence();
}

// One row of the encryption of the current item, by the whole workgroup: v pk + e of polynomial
// POLY of limb l, plus, on polynomial 0, the encodings rint(fv cos) of the value and
// rint(fb cos) of the brightness, written to `row`.  A wave's loads and stores complete in order,
// so a load issued after stores waits for them; therefore the first quarter of the keys comes
// loaded by the caller, the second half of the results is left to be stored by the next row
// (res, to `before` unless that is NULL) once its own keys are on their way, and the first half is
// stored when no load of this row is left.
template <int LOGN, int RC, int POLY, bool BRIGHT>
__device__ __forceinline__ void encrypt_row(RowHalf &res, uint64_t *before, uint64_t *row, const KeyPart &first, int l,
                                            int L, const double (&v)[1][2][16], double *lds, const Samples<LOGN> &smp,
                                            int B, double fv, double fb, const LimbConsts &lc, const DevTables &dt) {
  using F = Fft<LOGN>;
  constexpr double unit = Split<RC>::unit;
  const int tid = opaque(threadIdx.x);
  double x[2][2][16];  // low and high piece
  row_product(x, v, first, 0);
  {
    const Cplx *key = key_row<LOGN>(POLY, l, L, dt);
    const KeyPart k1 = load_part<LOGN>(key, 1), k2 = load_part<LOGN>(key, 2);
    stage_fence();
    row_product(x, v, k1, 1);
    const KeyPart k3 = load_part<LOGN>(key, 3);
    stage_fence();
    if (before) store_half<LOGN>(before, res, 1);
    row_product(x, v, k2, 2);
    row_product(x, v, k3, 3);
  }
  // The twist of value r is (cos, cos) of coefficients j and j + M, the factors of the encodings
  // as well: polynomial 0 loads them all, polynomial 1 forms them from the first.
  const int p = (int)fft_place<LOGN>((unsigned)opaque(threadIdx.x));
  Cplx t[POLY == 0 ? 16 : 1];
  auto load_twist = [&](int r) {
    return Cplx{*row_at(dt.cosj + F::T * r, (unsigned)p), *row_at(dt.cosj + F::M + F::T * r, (unsigned)p)};
  };
  fft_inverse<LOGN, 2>(x, lds, tid, dt.fft_inv, [&] {
    t[0] = load_twist(0);
    if constexpr (POLY == 0) {
#pragma unroll
      for (int r = 1; r < 4; r++) t[r] = load_twist(r);
    }
  });
  const double q = lc.q[l], qinv = lc.qinv[l], qinv_u = qinv * unit, b = (double)B;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    if constexpr (POLY == 0) {
      if (r % 4 == 0 && r < 8) {  // the next four, and before the first stores all
#pragma unroll
        for (int i = 4; i < (r == 4 ? 12 : 8); i++) t[(r + i) % 16] = load_twist(r + i);
        stage_fence();
      }
    }
    Cplx tw;
    if constexpr (POLY == 0)
      tw = t[r];
    else
      tw = fft_twist(t[0], r);
#pragma unroll
    for (int im = 0; im < 2; im++) {
      const double tr = im ? tw.im : tw.re, ti = im ? tw.re : -tw.im;
      // the error with its offset B, and the encodings, join the low piece before it is rounded
      double add = (double)((smp.at(r + 16 * im, p) >> (POLY == 0 ? kSmpShiftG2 : kSmpShiftG3)) & 0x7fu);
      if constexpr (POLY == 0) {
        add += __builtin_rint(fv * tr);
        if (BRIGHT) add += __builtin_rint(fb * tr);
      }
      const double lo = __builtin_fma(tr, x[0][0][r], __builtin_fma(ti, x[0][1][r], add));
      const double hi = __builtin_rint(__builtin_fma(tr, x[1][0][r], ti * x[1][1][r]));
      uint64_t w = encrypt_residue<LOGN, RC, POLY>(hi, lo, q, qinv, qinv_u, b);
      computed_here(w);
      res.w[im][r % 8] = w;
    }
    stage_fence();
    if (r == 7) store_half<LOGN>(row, res, 0);
  }
}

// All rows of the current item (its samples are drawn and v transformed).
template <int LOGN, int RC, bool BRIGHT>
__device__ __forceinline__ void encrypt_rows(int L, const double (&v)[1][2][16], double *lds, const Samples<LOGN> &smp,
                                             int B, double fv, double fb, uint64_t *out, const LimbConsts &lc,
                                             const DevTables &dt) {
  constexpr int N = 1 << LOGN;
  KeyPart first = load_part<LOGN>(key_row<LOGN>(0, 0, L, dt), 0);
  RowHalf res;
  uint64_t *before = nullptr;
#pragma unroll 1
  for (int l = 0; l < L; l++) {
    uint64_t *row0 = out + (size_t)l * N, *row1 = out + ((size_t)L + l) * N;
    encrypt_row<LOGN, RC, 0, BRIGHT>(res, before, row0, first, l, L, v, lds, smp, B, fv, fb, lc, dt);
    first = load_part<LOGN>(key_row<LOGN>(1, l, L, dt), 0);
    encrypt_row<LOGN, RC, 1, BRIGHT>(res, row0, row1, first, l, L, v, lds, smp, B, fv, fb, lc, dt);
    before = row1;
    first = load_part<LOGN>(key_row<LOGN>(0, l + 1 < L ? l + 1 : l, L, dt), 0);
  }
  store_half<LOGN>(before, res, 1);
}

// Bound by VALU issue and, nearly as much, by LDS stores: 65,536 encryptions at N = 8192 and 4 primes
// take 17.2 ms (3.8 M ciphertexts/s, 2 TB/s of stores) where 12 prime-field transforms took 23.7.
// About 2 ms of it are the samples, 1.5 the keys' loads and the stores.  Registers are budgeted for
// two waves per SIMD, that is two 256-thread workgroups per CU, of which one computes while the
// other waits; v_hat stays in 64 of them through all rows (reloaded for each row it took 20.8 ms).
// Other rings, 65,536 ciphertexts, before and now: N = 4096 7.26 and 6.36, N = 2048 3.31 and 3.00,
// N = 16384 92.6 and 68.9 ms.
template <int LOGN, int RC, int MODE, bool BRIGHT>
__global__ void __launch_bounds__(1 << (LOGN - 5)) __attribute__((amdgpu_waves_per_eu(2)))
    k_encrypt(EncJob job, const LimbConsts *__restrict__ lcp, DevTables dt) {
  constexpr int N = 1 << LOGN;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  const int L = lc.L, B = lc.B;
  const uint64_t count = enc_count<MODE>(job);
  for (uint64_t it = blockIdx.x; it < count; it += gridDim.x) {
    const EncItem e = enc_item<MODE, BRIGHT>(job, it, lc);
    Samples<LOGN> smp;
    draw_item<LOGN>(smp, lds, B, job.seed0, job.seed1, e.t, Fft<LOGN>::T, true, true, dt);
    double v[1][2][16];
    encrypt_forward<LOGN>(v, lds, smp, dt);
    encrypt_rows<LOGN, RC, BRIGHT>(L, v, lds, smp, B, e.fv, e.fb, job.out + e.slot * (uint64_t)(2 * L) * N, lc, dt);
  }
}

// The same for so few pixels that whole ciphertexts leave the device part empty: workgroup (i, p)
// encrypts rows p 2L/P..(p+1) 2L/P-1 of pixel i, P = gridDim.y (row w: polynomial w / L of limb w
// mod L).  Each draws the samples its rows need with all its threads, of which the first T stay
// for the transforms.
template <int LOGN, int RC, int MODE, bool BRIGHT>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2)))
    k_encrypt_few(EncJob job, const LimbConsts *__restrict__ lcp, DevTables dt) {
  constexpr int N = 1 << LOGN;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  const int L = lc.L, B = lc.B, item = (int)blockIdx.x, part = (int)blockIdx.y, parts = (int)gridDim.y;
  const int w0 = 2 * L * part / parts, w1 = 2 * L * (part + 1) / parts;
  if ((uint64_t)item >= enc_count<MODE>(job)) return;
  const EncItem e = enc_item<MODE, BRIGHT>(job, (uint64_t)item, lc);
  Samples<LOGN> smp;
  draw_item<LOGN>(smp, lds, B, job.seed0, job.seed1, e.t, (int)blockDim.x, w0 < L, w1 > L, dt);
  if (threadIdx.x >= Fft<LOGN>::T) return;  // whole waves: the barriers below are among the remaining ones
  double v[1][2][16];
  encrypt_forward<LOGN>(v, lds, smp, dt);
  uint64_t *out = job.out + e.slot * (uint64_t)(2 * L) * N, *before = nullptr;
  RowHalf res;
#pragma unroll 1
  for (int w = w0; w < w1; w++) {
    const int p = w >= L, l = p ? w - L : w;
    uint64_t *row = out + (size_t)w * N;
    const KeyPart first = load_part<LOGN>(key_row<LOGN>(p, l, L, dt), 0);
    if (p == 0)
      encrypt_row<LOGN, RC, 0, BRIGHT>(res, before, row, first, l, L, v, lds, smp, B, e.fv, e.fb, lc, dt);
    else
      encrypt_row<LOGN, RC, 1, BRIGHT>(res, before, row, first, l, L, v, lds, smp, B, e.fv, e.fb, lc, dt);
    before = row;
  }
  store_half<LOGN>(before, res, 1);
}

// ---------------------------------------------------------------------------
// The same through prime-field transforms, for N <= 8192: x = NTT(v) per limb, c0 =
// INTT(x pk0^) + e0 + m, c1 = INTT(x pk1^) + e1.  N/8 threads per ciphertext where the complex
// transforms have N/32, so it has the lower latency where whole ciphertexts just fill the device
// (encrypt_kernel in routes.hpp).  Compiled in units of its own, which a program that never takes it
// does not load.
// ---------------------------------------------------------------------------
// One limb of the encryption of the current item, by the whole workgroup (the samples are drawn: in
// smpl or, where they do not fit LDS, in smp).  With KEEP the canonical values of c0 and c1 are also
// returned in k0 and k1 (first-pass layout: register r holds coefficient tid + T r).
template <int LOGN, int LOGR, int RC, bool BRIGHT, bool KEEP>
__device__ __forceinline__ void encrypt_limb_ntt(int l, double *lds, const uint16_t *smpl,
                                                 const uint32_t (&smp)[1 << LOGR], int L, int B, double fv, double fb,
                                                 uint64_t *out, const LimbConsts &lc, const DevTables &dt,
                                                 double (&k0)[1 << LOGR], double (&k1)[1 << LOGR]) {
  using S = Shape<LOGN, LOGR>;
  using Red = Schedule<LOGN, RC>;
  constexpr int N = S::N, R = S::R, T = S::T;
  const double q = lc.q[l], qinv = lc.qinv[l];
  const int tid = opaque(threadIdx.x);
  auto sample = [&](int r) -> uint32_t {
    if constexpr (S::kSmpLds)
      return (uint32_t)smpl[tid + T * r];
    else
      return smp[r];
  };
  double x[R];
#pragma unroll
  for (int r = 0; r < R; r++) x[r] = (double)smp_t(sample(r));
  ntt_forward<LOGN, LOGR, Red::fwd_small>(x, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
  // both pointwise products at once (one wait for the key loads; x is then dead and
  // the second product takes its registers through the first inverse transform)
  double y[R], y1[R];
  const double *pk0 = dt.pk_hat + (size_t)l * N, *pk1 = dt.pk_hat + ((size_t)L + l) * N;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const unsigned e = elem_index<LOGN, LOGR, S::LAST>(tid, r);
    y[r] = mulmod(x[r], ld_table(pk0, e), q, qinv);
    y1[r] = mulmod(x[r], ld_table(pk1, e), q, qinv);
  }
  // the plaintext (and the brightness) and e0 of coefficient tid + T r
  auto message = [&](int r) {
    const double cs = ld_table(dt.cosj, tid + T * r);
    double m = (double)smp_g(sample(r), kSmpShiftG2, B) + __builtin_rint(fv * cs);
    if (BRIGHT) m += __builtin_rint(fb * cs);
    return m;
  };
  if constexpr (S::kDual) {
    // c0 and c1 of this limb through one paired inverse transform; the plaintext and
    // e0 are loaded before its final exchange
    double add[R];
    ntt_inverse2<LOGN, LOGR, Red::inv>(y, y1, lds, lds + S::SLOTS + kCdtSlots + 64, tid, dt.tw_inv + (size_t)l * N, q,
                                       qinv, [&] {
#pragma unroll
      for (int r = 0; r < R; r++) add[r] = message(r);
    });
    uint64_t *dst0 = out + (size_t)l * N, *dst1 = out + ((size_t)L + l) * N;
#pragma unroll
    for (int r = 0; r < R; r++) {
      const unsigned c = tid + T * r;
      const double v0 = canon(y[r] + add[r], q, qinv);
      const double v1 = canon(y1[r] + (double)smp_g(sample(r), kSmpShiftG3, B), q, qinv);
      __builtin_nontemporal_store(f64_to_u64(v0), word_at(dst0, c));
      __builtin_nontemporal_store(f64_to_u64(v1), word_at(dst1, c));
      if constexpr (KEEP) {
        k0[r] = v0;
        k1[r] = v1;
      }
    }
  } else {
#pragma unroll 1
    for (int poly = 0; poly < 2; poly++) {
      if (poly == 1) {
#pragma unroll
        for (int r = 0; r < R; r++) y[r] = y1[r];
      }
      double add[R];  // loaded before the final exchange
      ntt_inverse<LOGN, LOGR, Red::inv>(y, lds, tid, dt.tw_inv + (size_t)l * N, q, qinv, [&] {
#pragma unroll
        for (int r = 0; r < R; r++)
          add[r] = poly == 0 ? message(r) : (double)smp_g(sample(r), kSmpShiftG3, B);
      });
      uint64_t *dst = out + ((size_t)poly * L + l) * N;
#pragma unroll
      for (int r = 0; r < R; r++) {
        const double v = canon(y[r] + add[r], q, qinv);
        __builtin_nontemporal_store(f64_to_u64(v), word_at(dst, tid + T * r));
        if constexpr (KEEP) (poly == 0 ? k0 : k1)[r] = v;
      }
    }
  }
}

template <int LOGN, int LOGR, int RC, int MODE, bool BRIGHT>
__global__ void __launch_bounds__(1 << (LOGN - LOGR))
    k_encrypt_ntt(EncJob job, const LimbConsts *__restrict__ lcp, DevTables dt) {
  using S = Shape<LOGN, LOGR>;
  constexpr int N = S::N, T = S::T;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  uint64_t *cdt = reinterpret_cast<uint64_t *>(lds + S::SLOTS);
  uint16_t *smpl = reinterpret_cast<uint16_t *>(reinterpret_cast<char *>(lds) + S::enc_smp_at);
  uint8_t *guide = reinterpret_cast<uint8_t *>(lds) + S::enc_lds_bytes;
  const int tid = threadIdx.x;
  for (int i = tid; i < kCdtSlots; i += T) cdt[i] = dt.cdt[i];
  if constexpr (S::enc_guide != 0)
    for (int i = tid; i < (1 << S::enc_guide) / 8; i += T) reinterpret_cast<uint64_t *>(guide)[i] = dt.cdt[kCdtSlots + i];
  const int L = lc.L, B = lc.B;
  const uint64_t count = enc_count<MODE>(job);
  for (uint64_t it = blockIdx.x; it < count; it += gridDim.x) {
    const EncItem e = enc_item<MODE, BRIGHT>(job, it, lc);
    __syncthreads();
    draw_samples<LOGN, S::enc_guide != 0>(smpl, cdt, B, opaque(tid), T, job.seed0, job.seed1, e.t, kTagV, kTagE0, kTagE1, true, true,
                             guide);
    const uint32_t unused[S::R] = {};
    double k0[S::R], k1[S::R];
    for (int l = 0; l < L; l++)
      encrypt_limb_ntt<LOGN, LOGR, RC, BRIGHT, false>(l, lds, smpl, unused, L, B, e.fv, e.fb,
                                                      job.out + e.slot * (uint64_t)(2 * L) * N, lc, dt, k0, k1);
  }
}

// ---------------------------------------------------------------------------
// key generation, one workgroup per limb l: pk0_l = -a_l * s + e, pk1_l = a_l
// ---------------------------------------------------------------------------
template <int LOGN, int LOGR, int RC>
__global__ void __launch_bounds__(1 << (LOGN - LOGR))
    k_keygen(uint64_t k0, uint64_t k1, const LimbConsts *__restrict__ lcp, DevTables dt) {
  using S = Shape<LOGN, LOGR>;
  using Red = Schedule<LOGN, RC>;
  constexpr int N = S::N, R = S::R, T = S::T;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  uint64_t *cdt = reinterpret_cast<uint64_t *>(lds + S::SLOTS);
  uint16_t *lds16 = reinterpret_cast<uint16_t *>(lds);
  const int tid = threadIdx.x;
  for (int i = tid; i < kCdtSlots; i += T) cdt[i] = dt.cdt[i];
  __syncthreads();
  const int L = lc.L, B = lc.B, l = blockIdx.x;
  const double q = lc.q[l], qinv = lc.qinv[l];
  const uint64_t qi = lc.qi[l];
  uint32_t smp[R];
  // s from tag 16 (ternary), e from tag 17 (Gaussian); the third stream is unused
  draw_samples<LOGN, LOGR>(smp, lds16, cdt, B, tid, k0, k1, 0, kTagSk, kTagEk, kTagEk);
  // a_l: uniform residues by rejection, coefficient j tries block j, then N + j, ...
  // accept w < q * floor(2^64 / q) = 2^64 - (2^64 mod q)
  const uint64_t limit = 0ULL - ((~0ULL % qi + 1) % qi);
  double a[R];
  uint64_t *pk1 = dt.pk + ((size_t)L + l) * N;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const uint32_t j = (uint32_t)(tid + T * r);
    uint64_t val = 0;
    bool done = false;
    for (uint64_t att = 0; !done; att++) {
      const Philox4 w = philox4x64_10(0, kTagA0 + (uint32_t)l, att * N + j, 0, k0, k1);
#pragma unroll
      for (int k = 0; k < 4; k++) {
        if (!done && w.w[k] < limit) {
          val = w.w[k] % qi;
          done = true;
        }
      }
    }
    pk1[j] = val;
    a[r] = (double)val;
  }
  if (l == 0) {
#pragma unroll
    for (int r = 0; r < R; r++) dt.s[tid + T * r] = smp_t(smp[r]);
  }
  // s_hat * N^-1 for this limb
  double x[R];
#pragma unroll
  for (int r = 0; r < R; r++) x[r] = (double)smp_t(smp[r]);
  ntt_forward<LOGN, LOGR, Red::fwd_small>(x, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
  const double ninv = lc.ninv[l];
#pragma unroll
  for (int r = 0; r < R; r++) x[r] = reduce(mulmod(x[r], ninv, q, qinv), q, qinv);
  ntt_forward<LOGN, LOGR, Red::fwd_big>(a, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
#pragma unroll
  for (int r = 0; r < R; r++) a[r] = mulmod(a[r], x[r], q, qinv);
  ntt_inverse<LOGN, LOGR, Red::inv>(a, lds, tid, dt.tw_inv + (size_t)l * N, q, qinv);
  uint64_t *pk0 = dt.pk + (size_t)l * N;
#pragma unroll
  for (int r = 0; r < R; r++) {
    const double e = (double)smp_g(smp[r], kSmpShiftG2, B);
    pk0[tid + T * r] = (uint64_t)canon(e - a[r], q, qinv);
  }
}

// ---------------------------------------------------------------------------
// transforms of the keys, by one launch of 7 L + 1 workgroups
// ---------------------------------------------------------------------------
// A complex transform, times 1/M (fft.hpp), value r of thread tid at r T + tid: i = -1: s; 2 row +
// piece: the low or high piece of row p L + l, pk_p in limb l (centered residues).
template <int LOGN, int RC>
__device__ __forceinline__ void prepare_complex(int i, double *lds, const LimbConsts &lc, const DevTables &dt) {
  using F = Fft<LOGN>;
  constexpr double unit = Split<RC>::unit;
  const int tid = threadIdx.x, p = (int)fft_place<LOGN>((unsigned)tid), row = i >> 1;
  double x[1][2][16];
#pragma unroll
  for (int r = 0; r < 32; r++) {
    const int j = p + F::T * r;
    double v;
    if (i < 0) {
      v = (double)dt.s[j];
    } else {
      const double q = lc.q[row % lc.L], w = (double)dt.pk[(size_t)row * 2 * F::M + j];
      const double c = w > 0.5 * q ? w - q : w, hi = __builtin_rint(c * (1.0 / unit));
      v = i & 1 ? hi : __builtin_fma(-hi, unit, c);
    }
    x[0][r >> 4][r & 15] = v;
  }
  fft_forward<LOGN, 1>(x, lds, tid, dt.fft_fwd);
  Cplx *dst = i < 0 ? dt.s_fft : dt.pk_fft + (size_t)i * F::M;
#pragma unroll
  for (int r = 0; r < 16; r++) dst[r * F::T + tid] = Cplx{x[0][0][r] * (1.0 / F::M), x[0][1][r] * (1.0 / F::M)};
}

// Prime-field transforms, times N^-1, in limb l: which = 0: s; 1, 2: pk0, pk1.
template <int LOGN, int LOGR, int RC>
__device__ __forceinline__ void prepare_ntt(int l, int which, double *lds, const LimbConsts &lc, const DevTables &dt) {
  using S = Shape<LOGN, LOGR>;
  using Red = Schedule<LOGN, RC>;
  constexpr int N = S::N, R = S::R, T = S::T;
  const int tid = threadIdx.x, L = lc.L;
  const double q = lc.q[l], qinv = lc.qinv[l];
  double x[R];
  if (which == 0) {
#pragma unroll
    for (int r = 0; r < R; r++) x[r] = (double)dt.s[tid + T * r];
    ntt_forward<LOGN, LOGR, Red::fwd_small>(x, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
  } else {
    const uint64_t *src = dt.pk + ((size_t)(which - 1) * L + l) * N;
#pragma unroll
    for (int r = 0; r < R; r++) x[r] = (double)src[tid + T * r];
    ntt_forward<LOGN, LOGR, Red::fwd_big>(x, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
  }
  double *dst = which == 0 ? dt.s_hat + (size_t)l * N : dt.pk_hat + ((size_t)(which - 1) * L + l) * N;
#pragma unroll
  for (int r = 0; r < R; r++)
    dst[elem_index<LOGN, LOGR, S::LAST>(tid, r)] = reduce(mulmod(x[r], lc.ninv[l], q, qinv), q, qinv);
}

// Workgroups of the prime-field transforms' size, at most 512 threads; a complex transform takes the
// first T of them.
template <int LOGN>
constexpr int kPrepareLogr = LOGN == 14 ? 5 : 4;
template <int LOGN, int RC>
__global__ void __launch_bounds__(1 << (LOGN - kPrepareLogr<LOGN>)) __attribute__((amdgpu_waves_per_eu(2)))
    k_keys_prepare(const LimbConsts *__restrict__ lcp, DevTables dt) {
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  const int i = (int)blockIdx.x - 3 * lc.L;
  if (i < 0) {
    prepare_ntt<LOGN, kPrepareLogr<LOGN>, RC>((i + 3 * lc.L) % lc.L, (i + 3 * lc.L) / lc.L, lds, lc, dt);
  } else {
    if (threadIdx.x >= Fft<LOGN>::T) return;  // whole waves: the barriers below are among the remaining ones
    prepare_complex<LOGN, RC>(i - 1, lds, lc, dt);
  }
}

// ---------------------------------------------------------------------------
// launch helpers for one ring degree
// ---------------------------------------------------------------------------
template <auto KERNEL, size_t BYTES>
static hipError_t set_lds() {
  // once per kernel and device (also keeps the call out of graph captures after the first launch)
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 63;
  const uint64_t bit = 1ull << dev;
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(KERNEL),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)BYTES);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_acq_rel);
  return e;
}

}  // namespace ckks

#include "k_decrypt_impl.hpp"
#include "k_mul_impl.hpp"
#include "k_fused_impl.hpp"

namespace ckks {

// Kernels on complex transforms.
template <int LOGN, int RC>
struct FftLaunch {
  static constexpr int T = Fft<LOGN>::T;
  using B = FftLds<LOGN>;
  template <int MODE, bool BRIGHT>
  static hipError_t encrypt_as(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {
    hipError_t e = set_lds<k_encrypt<LOGN, RC, MODE, BRIGHT>, B::encrypt>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_encrypt<LOGN, RC, MODE, BRIGHT>), dim3((uint32_t)grid), dim3(T), B::encrypt, st, job, c->d_lc,
                       c->dev);
    return hipGetLastError();
  }
  // Workgroups as large as still leave two parts per pixel resident (8 waves per CU), then as many
  // parts as are: threads for the samples first, since every part draws them again (64 pixels at N
  // = 8192: 4 parts of 512 threads 42.6 us, 8 of 256 51.2).
  template <int MODE, bool BRIGHT>
  static hipError_t encrypt_few(const ckks_ctx *c, const EncJob &job, hipStream_t st) {
    hipError_t e = set_lds<k_encrypt_few<LOGN, RC, MODE, BRIGHT>, B::encrypt>();
    if (e != hipSuccess) return e;
    const uint64_t lanes = 512 * (uint64_t)c->num_cus;
    int threads = 512;
    while (threads > T && 2 * job.n * threads > lanes) threads /= 2;
    const uint64_t parts = std::min<uint64_t>(2 * c->lc.L, std::max<uint64_t>(1, lanes / threads / job.n));
    hipLaunchKernelGGL((k_encrypt_few<LOGN, RC, MODE, BRIGHT>), dim3((uint32_t)job.n, (uint32_t)parts), dim3(threads),
                       B::encrypt, st, job, c->d_lc, c->dev);
    return hipGetLastError();
  }
  static hipError_t prepare(const ckks_ctx *c, hipStream_t st) {
    using S = Shape<LOGN, kPrepareLogr<LOGN>>;
    hipError_t e = set_lds<k_keys_prepare<LOGN, RC>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_keys_prepare<LOGN, RC>), dim3(7 * c->lc.L + 1), dim3(S::T), S::lds_bytes, st, c->d_lc, c->dev);
    return hipGetLastError();
  }
  template <int LOGR, int LIMBS>
  static hipError_t decrypt_as(const ckks_ctx *c, const DecJob &job, uint64_t grid, hipStream_t st) {
    hipError_t e = set_lds<k_decrypt<LOGN, LOGR, RC, LIMBS>, B::exchange>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_decrypt<LOGN, LOGR, RC, LIMBS>), dim3((uint32_t)grid), dim3(T), B::exchange, st, job, c->d_lc,
                       c->dev);
    return hipGetLastError();
  }
  template <int LOGR>
  static hipError_t decrypt(const ckks_ctx *c, const DecJob &job, int limbs, uint64_t grid, hipStream_t st) {
    return limbs == 2 ? decrypt_as<LOGR, 2>(c, job, grid, st) : decrypt_as<LOGR, 1>(c, job, grid, st);
  }
};

// Kernels on prime-field transforms.
template <int LOGN, int LOGR, int RC>
struct Launch {
  using S = Shape<LOGN, LOGR>;
  using OnFft = FftLaunch<LOGN, RC>;
  static constexpr int kLogr = LOGR;
  static hipError_t keygen(const ckks_ctx *c, uint64_t s0, uint64_t s1, hipStream_t st) {
    hipError_t e = set_lds<k_keygen<LOGN, LOGR, RC>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_keygen<LOGN, LOGR, RC>), dim3(c->lc.L), dim3(S::T), S::lds_bytes, st, s0, s1, c->d_lc, c->dev);
    return hipGetLastError();
  }
  template <int MODE, bool BRIGHT>
  static hipError_t encrypt_as(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {
    hipError_t e = set_lds<k_encrypt_ntt<LOGN, LOGR, RC, MODE, BRIGHT>, S::enc_guided_lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_encrypt_ntt<LOGN, LOGR, RC, MODE, BRIGHT>), dim3((uint32_t)grid), dim3(S::T),
                       S::enc_guided_lds_bytes, st, job, c->d_lc, c->dev);
    return hipGetLastError();
  }
  template <int LIMBS>
  static hipError_t decrypt_as(const ckks_ctx *c, const DecJob &job, uint64_t grid, hipStream_t st) {
    hipError_t e = set_lds<k_decrypt_ntt<LOGN, LOGR, RC, LIMBS>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_decrypt_ntt<LOGN, LOGR, RC, LIMBS>), dim3((uint32_t)grid), dim3(S::T), S::lds_bytes, st, job,
                       c->d_lc, c->dev);
    return hipGetLastError();
  }
  static hipError_t decrypt(const ckks_ctx *c, const DecJob &job, int limbs, uint64_t grid, hipStream_t st) {
    return limbs == 2 ? decrypt_as<2>(c, job, grid, st) : decrypt_as<1>(c, job, grid, st);
  }
  template <bool DECRYPT, bool MISSES>
  static hipError_t fused_as(const ckks_ctx *c, const FusedJob &job, hipStream_t st) {
    constexpr auto kernel = k_cached_fused<LOGN, LOGR, RC, DECRYPT, MISSES>;
    constexpr size_t lds = MISSES ? S::enc_lds_bytes : DECRYPT ? S::lds_bytes : 0;
    hipError_t e = set_lds<kernel, lds>();
    if (e != hipSuccess) return e;
    // a persistent grid: the workgroups that fit on the device at once
    static std::atomic<int> resident{0};
    int g = resident.load(std::memory_order_relaxed);
    if (g == 0) {
      int per_cu = 0, cus = 0, dev = 0;
      e = hipGetDevice(&dev);
      if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void *>(kernel), S::T, lds);
      if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
      if (e != hipSuccess) return e;
      g = (per_cu < 1 ? 1 : per_cu) * (cus < 1 ? 1 : cus);
      resident.store(g, std::memory_order_relaxed);
    }
    uint64_t grid = job.n < (uint64_t)g ? job.n : (uint64_t)g;
    FusedJob jb = job;
    if (jb.ring) {  // each workgroup cycles through slots of its own: at most one per slot
      if (!jb.dec_out) return hipErrorInvalidValue;
      if (grid > jb.ring) grid = jb.ring;
    }
    if (!jb.counters) e = launch_fill_u32(jb.cursor, kXcds, 0u, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_cached_fused<LOGN, LOGR, RC, DECRYPT, MISSES>), dim3((uint32_t)grid), dim3(S::T), lds, st, jb,
                       c->d_lc, c->dev);
    return hipGetLastError();
  }
  static hipError_t fused(const ckks_ctx *c, const FusedJob &job, bool misses, hipStream_t st) {
    if (job.n == 0) return hipSuccess;
    if (!job.cursor || !job.seg_b || (misses ? !job.px : !job.counters)) return hipErrorInvalidValue;
    if (misses) return job.dec_out ? fused_as<true, true>(c, job, st) : fused_as<false, true>(c, job, st);
    return job.dec_out ? fused_as<true, false>(c, job, st) : fused_as<false, false>(c, job, st);
  }
  static hipError_t relin_keygen(const ckks_ctx *c, uint64_t s0, uint64_t s1, hipStream_t st) {
    hipError_t e = set_lds<k_relin_keygen<LOGN, LOGR, RC>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_relin_keygen<LOGN, LOGR, RC>), dim3(c->lc.L, c->lc.L + 1), dim3(S::T), S::lds_bytes, st, s0,
                       s1, c->d_lc, c->dev);
    return hipGetLastError();
  }
  static hipError_t relin_prepare(const ckks_ctx *c, hipStream_t st) {
    hipError_t e = set_lds<k_relin_prepare<LOGN, LOGR, RC>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_relin_prepare<LOGN, LOGR, RC>), dim3(c->lc.L, c->lc.L + 1, 2), dim3(S::T), S::lds_bytes, st,
                       c->d_lc, c->dev);
    return hipGetLastError();
  }
  template <bool SQUARE>
  static hipError_t mul_as(const ckks_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *out, uint64_t n, int level,
                           uint64_t *scratch, hipStream_t st) {
    hipError_t e = set_lds<k_mul<LOGN, LOGR, RC, SQUARE>, S::lds_bytes>();
    if (e != hipSuccess) return e;
    const uint64_t grid = n < kMulGroups ? n : kMulGroups;
    hipLaunchKernelGGL((k_mul<LOGN, LOGR, RC, SQUARE>), dim3((uint32_t)grid), dim3(S::T), S::lds_bytes, st, a, b, out, n,
                       level, scratch, c->d_lc, c->dev);
    return hipGetLastError();
  }
  static hipError_t mul(const ckks_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *out, uint64_t n, int level,
                        uint64_t *scratch, hipStream_t st) {
    return a == b ? mul_as<true>(c, a, b, out, n, level, scratch, st) : mul_as<false>(c, a, b, out, n, level, scratch, st);
  }
};

// The compiled form of an encryption kernel that a job takes: f(EncForm<mode, bright>).
template <int MODE, bool BRIGHT>
struct EncForm {
  static constexpr int mode = MODE;
  static constexpr bool bright = BRIGHT;
};
template <typename F>
static hipError_t encrypt_modes(const EncJob &job, F f) {
  const bool bright = job.seg_b != nullptr;
  if (job.vals || job.ts) {
    if (!job.vals || !job.ts || bright) return hipErrorInvalidValue;
    return f(EncForm<kEncEntries, false>{});
  }
  if (job.list) {
    if (!job.list_count) return hipErrorInvalidValue;
    return bright ? f(EncForm<kEncList, true>{}) : f(EncForm<kEncList, false>{});
  }
  if (job.list_count) return hipErrorInvalidValue;
  return bright ? f(EncForm<kEncPixels, true>{}) : f(EncForm<kEncPixels, false>{});
}

// All launchers of one ring degree, selecting the thread shape (where there is a choice) and the
// class of the primes (c->rc) at run time.
template <int LOGN>
struct RingLaunch {
  template <typename F>
  static hipError_t pick(const ckks_ctx *c, F f) {
    return c->rc ? f(FftLaunch<LOGN, 1>{}) : f(FftLaunch<LOGN, 0>{});
  }
  template <typename F>
  static hipError_t pick(const ckks_ctx *c, int logr, F f) {
    if constexpr (LOGN - 3 <= 10) {  // 8 values per thread: N/8 threads, at most 1024
      if (logr == 3) return c->rc ? f(Launch<LOGN, 3, 1>{}) : f(Launch<LOGN, 3, 0>{});
    }
    if (logr == 4) return c->rc ? f(Launch<LOGN, 4, 1>{}) : f(Launch<LOGN, 4, 0>{});
    if (logr == 5) return c->rc ? f(Launch<LOGN, 5, 1>{}) : f(Launch<LOGN, 5, 0>{});
    return hipErrorInvalidValue;
  }
  static hipError_t encrypt(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {
    if (job.n == 0) return hipSuccess;
    const int kernel = job.kernel >= 0 ? job.kernel : encrypt_kernel(LOGN, c->lc.L, job.n, (uint64_t)c->num_cus);
    if (kernel == kEncPrime && LOGN <= 13) return launch_encrypt_prime(c, job, grid, st);
    const bool split = kernel == kEncSplit && job.n <= grid;
    return encrypt_modes(job, [&](auto M) {
      return pick(c, [&](auto L) {
        using K = decltype(L);
        using E = decltype(M);
        return split ? K::template encrypt_few<E::mode, E::bright>(c, job, st)
                     : K::template encrypt_as<E::mode, E::bright>(c, job, grid, st);
      });
    });
  }
  static hipError_t encrypt_prime(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {
    return encrypt_modes(job, [&](auto M) {
      return pick(c, c->logr_enc, [&](auto L) {
        using E = decltype(M);
        return decltype(L)::template encrypt_as<E::mode, E::bright>(c, job, grid, st);
      });
    });
  }
  static hipError_t decrypt(const ckks_ctx *c, const DecJob &job, int limbs, uint64_t grid, hipStream_t st) {
    if constexpr (kDecryptFft<LOGN>)
      if (decrypt_complex(LOGN, c->rc, limbs, grid, (uint64_t)c->num_cus))
        return pick(c, c->logr_dec, [&](auto L) {
          using K = decltype(L);
          return K::OnFft::template decrypt<K::kLogr>(c, job, limbs, grid, st);
        });
    return pick(c, c->logr_dec, [&](auto L) { return decltype(L)::decrypt(c, job, limbs, grid, st); });
  }
};

}  // namespace ckks

// Define the per-ring-degree launcher entry points.  Each ring degree's kernels are spread
// over four translation units (k_ntt_<LOGN>_{enc,prime,mul,fused}.hip) so they compile in parallel
// and load when first used.
#define CKKS_DEFINE_RING_ENC(LOGN)                                                                                  \
  namespace ckks {                                                                                                  \
  hipError_t launch_encrypt_##LOGN(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {           \
    return RingLaunch<LOGN>::encrypt(c, job, grid, st);                                                             \
  }                                                                                                                 \
  hipError_t launch_keygen_##LOGN(const ckks_ctx *c, uint64_t s0, uint64_t s1, hipStream_t st) {                    \
    return RingLaunch<LOGN>::pick(c, c->logr_enc, [&](auto L) { return decltype(L)::keygen(c, s0, s1, st); });      \
  }                                                                                                                 \
  hipError_t launch_keys_prepare_##LOGN(const ckks_ctx *c, hipStream_t st) {                                        \
    return RingLaunch<LOGN>::pick(c, [&](auto L) { return decltype(L)::prepare(c, st); });                          \
  }                                                                                                                 \
  hipError_t launch_decrypt_##LOGN(const ckks_ctx *c, const DecJob &job, int limbs, uint64_t grid, hipStream_t st) { \
    return RingLaunch<LOGN>::decrypt(c, job, limbs, grid, st);                                                      \
  }                                                                                                                 \
  }

#define CKKS_DEFINE_RING_PRIME(LOGN)                                                                                \
  namespace ckks {                                                                                                  \
  hipError_t launch_encrypt_prime_##LOGN(const ckks_ctx *c, const EncJob &job, uint64_t grid, hipStream_t st) {     \
    return RingLaunch<LOGN>::encrypt_prime(c, job, grid, st);                                                       \
  }                                                                                                                 \
  }

#define CKKS_DEFINE_RING_MUL(LOGN)                                                                                  \
  namespace ckks {                                                                                                  \
  hipError_t launch_relin_keygen_##LOGN(const ckks_ctx *c, uint64_t s0, uint64_t s1, hipStream_t st) {              \
    return RingLaunch<LOGN>::pick(c, c->logr_mul, [&](auto L) { return decltype(L)::relin_keygen(c, s0, s1, st); });   \
  }                                                                                                                 \
  hipError_t launch_relin_prepare_##LOGN(const ckks_ctx *c, hipStream_t st) {                                       \
    return RingLaunch<LOGN>::pick(c, c->logr_mul, [&](auto L) { return decltype(L)::relin_prepare(c, st); });          \
  }                                                                                                                 \
  hipError_t launch_mul_##LOGN(const ckks_ctx *c, const uint64_t *a, const uint64_t *b, uint64_t *out, uint64_t n,  \
                               int level, uint64_t *scratch, hipStream_t st) {                                      \
    return RingLaunch<LOGN>::pick(                                                                                  \
        c, c->logr_mul, [&](auto L) { return decltype(L)::mul(c, a, b, out, n, level, scratch, st); });                \
  }                                                                                                                 \
  }

#define CKKS_DEFINE_RING_FUSED(LOGN)                                                                                \
  namespace ckks {                                                                                                  \
  hipError_t launch_cached_fused_##LOGN(const ckks_ctx *c, const FusedJob &job, bool misses, hipStream_t st) {       \
    return RingLaunch<LOGN>::pick(c, c->logr_dec, [&](auto L) { return decltype(L)::fused(c, job, misses, st); });  \
  }                                                                                                                 \
  }
