"""The last step of the complex-transform encryption, on the host: for every class of primes and both
polynomials, the quotient forms and the packing that the kernel compiles give the residues of
exact integer arithmetic, for random and extreme inputs; and the recombination of two pieces stays
within its bound at quotients close to a half."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2409_03568_amd", "csrc")
SRC = os.path.join(HERE, "native", "encrypt_emulation.cpp")
LIB = os.path.join(HERE, "native", "libencrypt_emulation.so")
DEPS = [SRC, os.path.join(HERE, "native", "fft_emulation.cpp")] + [
    os.path.join(CSRC, f) for f in ("fft.hpp", "ntt.hpp", "modarith.hpp", "philox.hpp", "host_math.cpp", "host_math.hpp")]


@pytest.fixture(scope="module")
def emu():
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    if not (os.path.exists(LIB) and os.path.getmtime(LIB) >= max(os.path.getmtime(d) for d in DEPS)):
        tmp = LIB + ".tmp%d" % os.getpid()
        subprocess.run([hipcc, "-x", "hip", "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-arch=gfx950",
                        "-ffp-contract=off", "-o", tmp, SRC, os.path.join(CSRC, "host_math.cpp")],
                       check=True, capture_output=True)
        os.replace(tmp, LIB)
    L = C.CDLL(LIB)
    d, u = C.POINTER(C.c_double), C.POINTER(C.c_uint64)
    L.emu_encrypt_row.argtypes = [C.c_int, d, u, C.c_uint64, C.c_int, C.c_int, C.POINTER(C.c_uint32), C.c_int, C.c_double,
                                  C.c_double, u]
    L.emu_combine.argtypes = [d, d, C.c_int, C.c_int, C.c_uint64, d, d]
    return L


def _p(a, t):
    return a.ctypes.data_as(C.POINTER(t))


@pytest.mark.parametrize("log_n,bits", [(11, 20), (11, 30), (11, 40), (11, 41), (11, 50), (12, 36), (12, 40), (12, 41),
                                        (12, 50), (13, 36), (13, 40), (13, 41), (13, 50), (14, 36), (14, 40), (14, 41),
                                        (14, 50)])
def test_rows_are_exact(emu, oracle_mod, log_n, bits):
    N, rc, B = 1 << log_n, 0 if bits <= 40 else 1, 63
    rng = np.random.default_rng([log_n, bits])
    q = oracle_mod.gen_primes(log_n, bits, 1)[0]
    psi = oracle_mod.primitive_2n_root(q, log_n)
    cos = np.cos(np.pi * np.arange(N) / N)
    uniform = rng.integers(0, q, N, dtype=np.uint64)
    ternary = rng.integers(-1, 2, N)
    noise = rng.integers(-B, B + 1, N)
    largest = 255.0 * 2.0 ** (int(np.floor(np.log2(q))) - 8)     # 256 2^(scale + 1 - log N) below the prime
    cases = [("random", ternary, uniform, noise, largest / 2**12, 0.0),
             ("largest value", ternary, uniform, noise, largest, 0.0),
             ("largest brightness", ternary, uniform, noise, largest, -(2.0**50 - 2.0**10)),
             ("no message", ternary, uniform, noise, 0.0, 0.0),
             ("zero key", ternary, np.zeros(N, dtype=np.uint64), noise, 0.0, 0.0),      # residues next to 0 and q
             ("ones x half", np.ones(N, dtype=np.int64), np.full(N, q // 2, dtype=np.uint64), noise, largest, 0.0),
             ("ones x above half", np.ones(N, dtype=np.int64), np.full(N, q // 2 + 1, dtype=np.uint64), -noise, 0.0, 2.0**49),
             ("all noise high", np.zeros(N, dtype=np.int64), uniform, np.full(N, B), 0.0, 0.0),
             ("all noise low", np.zeros(N, dtype=np.int64), uniform, np.full(N, -B), 0.0, 0.0)]
    for name, v, wide, e, fv, fb in cases:
        prod = oracle_mod.negacyclic_mul(np.array([int(x) % q for x in v], dtype=np.uint64), wide, q, psi)
        for poly in (0, 1):
            m = np.rint(fv * cos) + np.rint(fb * cos) if poly == 0 else np.zeros(N)
            want = np.array([(int(prod[j]) + int(e[j]) + int(m[j])) % q for j in range(N)], dtype=np.uint64)
            got = np.zeros(N, dtype=np.uint64)
            vd, ev = np.ascontiguousarray(v, dtype=np.float64), (e + B).astype(np.uint32)
            assert emu.emu_encrypt_row(log_n, _p(vd, C.c_double), _p(wide, C.c_uint64), q, rc, poly, _p(ev, C.c_uint32), B,
                                       fv, fb, _p(got, C.c_uint64)) == 0
            assert np.array_equal(got, want), (name, poly, np.nonzero(got != want)[0][:5])


@pytest.mark.parametrize("bits", [36, 40, 41, 50])
@pytest.mark.parametrize("log_n", [11, 12, 13, 14])
def test_combine_near_half_quotients(emu, oracle_mod, log_n, bits):
    """|result| <= q/2 + N q 2^-51 + 1: the quotient, of magnitude up to N, is off by up to N 2^-51."""
    N, rc = 1 << log_n, 0 if bits <= 40 else 1
    h = 25 if rc else 20
    q = oracle_mod.gen_primes(log_n, bits, 1)[0]
    rng = np.random.default_rng([log_n, bits])
    top = N << max(bits - h, 1)                                   # |hi| of a canonical residue's high piece
    k = np.concatenate([rng.integers(-N, N, 4000), np.array([N - 1, N - 2, 1 - N, 0, -1])])
    reach = max(3, int(N * q * 2.0**-50))                         # twice the bound's excess over q/2
    off = rng.integers(-reach, reach + 1, len(k))
    total = [int(a) * q + q // 2 + int(b) for a, b in zip(k, off)]  # next to (k + 1/2) q
    hi = np.array([min(max((t + (1 << (h - 1))) >> h, -top), top) for t in total], dtype=np.int64)
    w = np.array([t - (int(x) << h) for t, x in zip(total, hi)], dtype=object)
    keep = [abs(int(x)) < N << h for x in w]
    hi, w, total = hi[keep], w[keep], [t for t, s in zip(total, keep) if s]
    assert len(total) > 1000
    hd, wd = hi.astype(np.float64), np.array([float(x) for x in w])
    out, cen = np.zeros(len(hd)), np.zeros(len(hd))
    emu.emu_combine(_p(hd, C.c_double), _p(wd, C.c_double), len(hd), rc, q, _p(out, C.c_double), _p(cen, C.c_double))
    bound = q / 2 + N * q * 2.0**-51 + 1
    assert np.abs(out).max() <= bound
    for r, c, t in zip(out, cen, total):
        assert (int(r) - t) % q == 0 and (int(c) - t) % q == 0 and 2 * abs(int(c)) < q
