// Decryption kernels (Sec. 2.2.2): c0 + c1 s through complex transforms (fft.hpp), the decode
// of slot 0, and the two-limb CRT lift.  Included by the transform implementation header, whose
// shapes and tables they use.
#pragma once

namespace ckks {

// ---------------------------------------------------------------------------
// decryption and decoding of slot 0:
//   d_i = c0_i + c1_i s mod q_i in limb i;  out = sum_j x_j cos(pi j/N) / scale
// LIMBS = 1: x_j is the centered residue of limb 0, exact while |x_j| < q_0/2.
// LIMBS = 2: x_j is the centered CRT lift of limbs 0 and 1, x = x0 + q_0 k with
//   x0 = [d_0]_{q_0} and k = [(d_1 - x0) q_0^-1]_{q_1}, exact while |x_j| < q_0 q_1 / 2
//   (the sum is formed in FP64, so a lift beyond 2^53 is rounded to 53 bits).
// ---------------------------------------------------------------------------
// x = c0 + x s mod q, |x| as of fft_combine, from integer-valued x in [0, 2^52) (c1; register r:
// coefficient p + T r) and c0(r), the canonical coefficient of the same register.  load(0) and
// load(1) run before the last pass and after it, for the c0 of values 0..7 and 8..15.
template <int LOGN, int RC, class LOAD, class C0>
__device__ __forceinline__ void times_s_plus(double (&c1)[32], double *lds, double q, double qinv, const DevTables &dt,
                                             LOAD &&load, C0 &&c0) {
  using F = Fft<LOGN>;
  constexpr double unit = Split<RC>::unit;
  const int tid = opaque(threadIdx.x);
  double x[2][2][16];  // low and high piece
#pragma unroll
  for (int r = 0; r < 32; r++) {
    const double hi = __builtin_rint(c1[r] * (1.0 / unit));
    x[0][r >> 4][r & 15] = __builtin_fma(-hi, unit, c1[r]);
    x[1][r >> 4][r & 15] = hi;
    computed_here(x[0][r >> 4][r & 15]);
    computed_here(x[1][r >> 4][r & 15]);
  }
  fft_forward<LOGN, 2>(x, lds, tid, dt.fft_fwd);
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const Cplx k = ld_row(dt.s_fft + r * F::T, (unsigned)tid);
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const double xr = x[i][0][r], xi = x[i][1][r];
      x[i][0][r] = __builtin_fma(xr, k.re, -(xi * k.im));
      x[i][1][r] = __builtin_fma(xr, k.im, xi * k.re);
      computed_here(x[i][0][r]);
      computed_here(x[i][1][r]);
    }
  }
  stage_fence();
  Cplx t0;
  fft_inverse<LOGN, 2>(x, lds, tid, dt.fft_inv, [&] {
    const unsigned p = fft_place<LOGN>((unsigned)opaque(threadIdx.x));
    t0 = Cplx{*row_at(dt.cosj, p), *row_at(dt.cosj + F::M, p)};
    load(0);
  });
  load(1);
  stage_fence();
  const double qinv_u = qinv * unit;
#pragma unroll
  for (int r = 0; r < 16; r++) {
    const Cplx t = fft_twist(t0, r);
#pragma unroll
    for (int im = 0; im < 2; im++) {
      const double tr = im ? t.im : t.re, ti = im ? t.re : -t.im;
      const double lo = __builtin_rint(__builtin_fma(tr, x[0][0][r], ti * x[0][1][r]));
      const double hi = __builtin_rint(__builtin_fma(tr, x[1][0][r], ti * x[1][1][r]));
      c1[r + 16 * im] = fft_combine(hi, lo + c0(r + 16 * im), unit, q, qinv, qinv_u);
      computed_here(c1[r + 16 * im]);
    }
    stage_fence();
  }
}

// A row of a ciphertext in coefficient order (register r: coefficient p + T r).
template <int LOGN>
__device__ __forceinline__ void load_row(double (&x)[32], const uint64_t *row) {
  const unsigned p = fft_place<LOGN>((unsigned)opaque(threadIdx.x));
#pragma unroll
  for (int r = 0; r < 32; r++) x[r] = u64_to_f64(__builtin_nontemporal_load(row_at(row + Fft<LOGN>::T * r, p)));
}

// d = c0 + c1 s mod q, |d| as of fft_combine, in coefficient order: c1 in x (consumed), c0 in memory.
template <int LOGN, int RC>
__device__ __forceinline__ void decrypt_limb(double (&x)[32], const uint64_t *c0, double *lds, double q, double qinv,
                                             const DevTables &dt) {
  constexpr int T = Fft<LOGN>::T;
  uint64_t c0w[32];
  times_s_plus<LOGN, RC>(
      x, lds, q, qinv, dt,
      [&](int h) {
        const unsigned p = fft_place<LOGN>((unsigned)opaque(threadIdx.x));
#pragma unroll
        for (int i = 0; i < 16; i++) {
          const int r = 8 * h + (i & 7) + 16 * (i >> 3);
          c0w[r] = __builtin_nontemporal_load(row_at(c0 + T * r, p));
        }
      },
      [&](int r) { return u64_to_f64(c0w[r]); });
}

// sum_j x_j cos(pi j / N) over the workgroup, returned in thread 0, in the order of the prime-field
// kernel with 2^LOGR values per thread, so that a ciphertext's decoded value does not depend on
// which kernel a call takes: TC = N / 2^LOGR chains j = i mod TC, each summed with increasing j,
// combined by butterflies over 64 consecutive chains and then in sequence.  sums: the exchange space.
template <int LOGN, int LOGR>
__device__ __forceinline__ double slot0_sum(const double (&x)[32], double *sums, const DevTables &dt) {
  constexpr int T = Fft<LOGN>::T, TC = 1 << (LOGN - LOGR), A = TC / T;  // chains per thread
  const int tid = opaque(threadIdx.x);
  const unsigned p = fft_place<LOGN>((unsigned)tid);
  double acc[A];
#pragma unroll
  for (int a = 0; a < A; a++) acc[a] = 0.0;
#pragma unroll
  for (int r = 0; r < 32; r++) acc[r % A] = __builtin_fma(x[r], *row_at(dt.cosj + T * r, p), acc[r % A]);
  __syncthreads();  // every wave has read the exchange space
#pragma unroll
  for (int a = 0; a < A; a++) sums[p + T * a] = acc[a];
  __syncthreads();
#pragma unroll
  for (int a = 0; a < A; a++) {
    acc[a] = sums[tid + T * a];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc[a] += __shfl_xor(acc[a], off, 64);
  }
  double *waves = sums + TC;
#pragma unroll
  for (int a = 0; a < A; a++)
    if ((tid & 63) == 0) waves[(tid >> 6) + a * (T / 64)] = acc[a];
  __syncthreads();
  double s = 0.0;
  if (tid == 0)
    for (int w = 0; w < TC / 64; w++) s += waves[w];
  return s;
}

// Ciphertext of item i of a decryption (a position in the list, if there is one).
struct DecItem {
  uint64_t slot, item;
};
__device__ __forceinline__ uint64_t dec_count(const DecJob &job) {
  if (!job.list) return job.n;
  if (!gate_open(job.gate, job.list_count)) return 0;
  const uint64_t m = *job.list_count;
  const uint64_t left = m > job.list_first ? m - job.list_first : 0;
  return left < job.n ? left : job.n;
}
__device__ __forceinline__ DecItem dec_item(const DecJob &job, uint64_t i) {
  if (!job.list) return DecItem{i, i};
  const uint64_t item = job.list[job.list_first + i];
  return DecItem{job.compact ? i : item, item};
}

// Registers are budgeted for two waves per SIMD; the two-limb form holds limb 0's values across
// limb 1's transforms (32 registers spilled; with the limbs side by side in one workgroup of
// twice the threads nothing is spilled, but all of them wait for each other: 8.5 against 6.8 ms
// per 65,536 at N = 8192).  LOGR: the order of the decoded sum only.
template <int LOGN, int LOGR, int RC, int LIMBS>
__global__ void __launch_bounds__(1 << (LOGN - 5)) __attribute__((amdgpu_waves_per_eu(2)))
    k_decrypt(DecJob job, const LimbConsts *__restrict__ lcp, DevTables dt) {
  constexpr int N = 1 << LOGN;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  const double q = lc.q[0];
  const uint64_t n = dec_count(job);
  for (uint64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const DecItem it = dec_item(job, i);
    const uint64_t *c0 = job.cts + it.slot * (uint64_t)(2 * job.level) * N;
    const uint64_t *c1 = c0 + (size_t)job.level * N;
    double x[32];
    load_row<LOGN>(x, c1);
    decrypt_limb<LOGN, RC>(x, c0, lds, q, lc.qinv[0], dt);
#pragma unroll
    for (int r = 0; r < 32; r++) {
      x[r] = wrap_center(x[r], q);
      computed_here(x[r]);
    }
    if constexpr (LIMBS == 2) {
      const double q1 = lc.q[1], q1inv = lc.qinv[1], w = lc.q0inv_q1;
      double y[32];
      load_row<LOGN>(y, c1 + N);
      decrypt_limb<LOGN, RC>(y, c0 + N, lds, q1, q1inv, dt);
#pragma unroll
      for (int r = 0; r < 32; r++) {
        // |y| < q_1/2 + 2^13 and |x| <= q_0/2: the difference stays below 2^51
        const double k = center(mulmod(y[r] - x[r], w, q1, q1inv), q1, q1inv);
        x[r] = __builtin_fma(k, q, x[r]);
        computed_here(x[r]);
      }
    }
    const double s = slot0_sum<LOGN, LOGR>(x, lds, dt);
    if (threadIdx.x == 0) job.out[it.item] = s * job.inv_scale;
  }
}

// ---------------------------------------------------------------------------
// The same through prime-field transforms (ntt.hpp), with 8 or 16 values per thread and so two to
// four times the waves.
// ---------------------------------------------------------------------------
// Which of the two decrypts: decrypt_complex in routes.hpp.
template <int LOGN>
constexpr bool kDecryptFft = LOGN == 13;

// Register budget: enough waves per SIMD for as many workgroups as the LDS admits on a
// CU (at most two), so one workgroup's waves compute while another's wait at a barrier.
template <int LOGN, int LOGR>
constexpr int decrypt_waves_per_eu() {
  constexpr int wgs = (int)((160 * 1024) / Shape<LOGN, LOGR>::lds_bytes) >= 2 ? 2 : 1;
  constexpr int w = wgs * (1 << (LOGN - LOGR)) / 256;
  return w < 1 ? 1 : w;
}
// The two-limb form holds limb 0's values across limb 1's transform: half the waves, so
// that they stay in registers (forcing the one-limb occupancy spills them to scratch,
// about 9 GiB of memory traffic per 65,536 ciphertexts, for 2% less time).
template <int LOGN, int LOGR, int LIMBS>
constexpr int decrypt_waves_hint() {
  constexpr int w = decrypt_waves_per_eu<LOGN, LOGR>() / LIMBS;
  return w < 1 ? 1 : w;
}

// d = c0 + c1 * s in limb l of ciphertext (c0, c1), returned in x in the first-pass
// layout as signed values below 2^52 in magnitude (congruent to d mod q_l).
template <int LOGN, int LOGR, int RC>
__device__ __forceinline__ void decrypt_limb_ntt(double (&x)[1 << LOGR], const uint64_t *c0, const uint64_t *c1, int l,
                                             double *lds, int tid, const LimbConsts &lc, const DevTables &dt) {
  using S = Shape<LOGN, LOGR>;
  using Red = Schedule<LOGN, RC>;
  constexpr int N = S::N, R = S::R, T = S::T;
  const double q = lc.q[l], qinv = lc.qinv[l];
  const uint64_t *c0l = c0 + (size_t)l * N, *c1l = c1 + (size_t)l * N;
#pragma unroll
  for (int r = 0; r < R; r++) x[r] = u64_to_f64(__builtin_nontemporal_load(word_at(c1l, tid + T * r)));
  ntt_forward<LOGN, LOGR, Red::fwd_big>(x, lds, tid, dt.tw_fwd + (size_t)l * N, q, qinv);
  const double *sh = dt.s_hat + (size_t)l * N;
#pragma unroll
  for (int r = 0; r < R; r++) x[r] = mulmod(x[r], ld_table(sh, elem_index<LOGN, LOGR, S::LAST>(tid, r)), q, qinv);
  // c0 is loaded from HBM before the final exchange of the transform
  uint64_t c0w[R];
  ntt_inverse<LOGN, LOGR, Red::inv>(x, lds, tid, dt.tw_inv + (size_t)l * N, q, qinv, [&] {
#pragma unroll
    for (int r = 0; r < R; r++) c0w[r] = __builtin_nontemporal_load(word_at(c0l, tid + T * r));
  });
#pragma unroll
  for (int r = 0; r < R; r++) x[r] += u64_to_f64(c0w[r]);
}

template <int LOGN, int LOGR, int RC, int LIMBS>
__global__ void __launch_bounds__(1 << (LOGN - LOGR))
    __attribute__((amdgpu_waves_per_eu(decrypt_waves_hint<LOGN, LOGR, LIMBS>())))
    k_decrypt_ntt(DecJob job, const LimbConsts *__restrict__ lcp, DevTables dt) {
  using S = Shape<LOGN, LOGR>;
  constexpr int N = S::N, R = S::R, T = S::T;
  const LimbConsts &lc = *lcp;
  extern __shared__ __attribute__((aligned(128))) double lds[];
  double *red = lds + S::SLOTS + kCdtSlots;
  const int tid = threadIdx.x;
  const double q = lc.q[0], qinv = lc.qinv[0];
  const uint64_t n = dec_count(job);
  for (uint64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int tid = opaque(threadIdx.x);
    const DecItem it = dec_item(job, i);
    const uint64_t *c0 = job.cts + it.slot * (uint64_t)(2 * job.level) * N;
    const uint64_t *c1 = c0 + (size_t)job.level * N;
    double x[R];
    decrypt_limb_ntt<LOGN, LOGR, RC>(x, c0, c1, 0, lds, tid, lc, dt);
#pragma unroll
    for (int r = 0; r < R; r++) x[r] = center(x[r], q, qinv);
    if constexpr (LIMBS == 2) {
      const double q1 = lc.q[1], q1inv = lc.qinv[1], w = lc.q0inv_q1;
      double y[R];
      decrypt_limb_ntt<LOGN, LOGR, RC>(y, c0, c1, 1, lds, tid, lc, dt);
#pragma unroll
      for (int r = 0; r < R; r++) {
        // |y| < 2^52 and |x| <= q_0/2: the difference of the reduced values stays below 2^51
        const double k = center(mulmod(reduce(y[r], q1, q1inv) - x[r], w, q1, q1inv), q1, q1inv);
        x[r] = __builtin_fma(k, q, x[r]);
      }
    }
    double acc = 0.0;
#pragma unroll
    for (int r = 0; r < R; r++) acc = __builtin_fma(x[r], ld_table(dt.cosj, tid + T * r), acc);
    // workgroup sum in a fixed order: wave butterflies, then the waves in sequence
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((tid & 63) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < T / 64; w++) s += red[w];
      job.out[it.item] = s * job.inv_scale;
    }
  }
}

}  // namespace ckks
