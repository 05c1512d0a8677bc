"""CPU checks of the complex transforms behind encryption and decryption, run through a host
emulation: the product of a ternary polynomial with a wide one, split into two pieces, equals
the oracle's product modulo the prime, every coefficient of a piece stays within the derived
bound of its integer, and the layouts (LDS slots, wave-local exchanges, key positions) hold
every element once.  Also the samplers' guide: the search through it gives the plain search's value
for every word that could tell them apart."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2409_03568_amd", "csrc")
SRC = os.path.join(HERE, "native", "fft_emulation.cpp")
LIB = os.path.join(HERE, "native", "libfft_emulation.so")
DEPS = [SRC] + [os.path.join(CSRC, f) for f in ("fft.hpp", "ntt.hpp", "modarith.hpp", "philox.hpp", "host_math.cpp",
                                                "host_math.hpp")]


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
    L.emu_fft_product.argtypes = [C.POINTER(C.c_double), C.POINTER(C.c_uint64), C.c_int, C.c_int, C.c_uint64, C.c_int,
                                  C.POINTER(C.c_uint64), C.POINTER(C.c_double)]
    L.emu_guide_mismatches.argtypes = [C.c_double, C.c_int, C.POINTER(C.c_uint64), C.c_int]
    return L


@pytest.mark.parametrize("sigma,B", [(3.2, 19), (0.5, 3), (1.0, 6), (3.2, 1), (8.0, 63), (10.0, 40)])
def test_gauss_guide(emu, sigma, B):
    w = np.random.default_rng(B).integers(0, 2**64, 200000, dtype=np.uint64)
    w[:2] = [0, 2**64 - 1]
    assert emu.emu_guide_mismatches(sigma, B, w.ctypes.data_as(C.POINTER(C.c_uint64)), len(w)) == 0


@pytest.mark.parametrize("log_n,bits", [(11, 20), (11, 30), (11, 49), (12, 36), (12, 40), (12, 50), (13, 40), (13, 41),
                                        (13, 50), (14, 36), (14, 50)])
def test_split_product_is_exact(emu, oracle_mod, log_n, bits):
    N, rc = 1 << log_n, 0 if bits <= 40 else 1
    rng = np.random.default_rng(log_n * 100 + bits)
    q = oracle_mod.gen_primes(log_n, bits, 1)[0]
    psi = oracle_mod.primitive_2n_root(q, log_n)
    alt = np.where(np.arange(N) % 2 == 0, 1, -1)
    uniform = rng.integers(0, q, N, dtype=np.uint64)
    h = 25 if rc else 20
    worst = np.uint64(min(q - 1, ((q >> 1 >> h) << h) + (1 << (h - 1)) - 1))  # both pieces near their largest
    # |small|_2 |piece|_2 <= 2^h N: the low piece is below 2^(h-1), the high one below 2^(bits-h)
    bound = 12 * 2.0**-53 * (3 * (log_n - 1) + 1) * 2.0**h * N
    for name, small, wide in [("random", rng.integers(-1, 2, N), uniform), ("ones", np.ones(N), uniform),
                              ("alternating", alt, np.full(N, q - 1, dtype=np.uint64)),
                              ("ones x largest", np.ones(N), np.full(N, worst)),
                              ("minus one x q - 1", -np.ones(N), np.full(N, q - 1, dtype=np.uint64)),
                              ("zero", np.zeros(N), uniform)]:
        s = np.ascontiguousarray(small, dtype=np.float64)
        ref = oracle_mod.negacyclic_mul(np.array([int(x) % q for x in small], dtype=np.uint64), wide, q, psi)
        for center in (0, 1):  # decryption splits the canonical residue, the key tables the centered one
            c, off = np.zeros(N, dtype=np.uint64), C.c_double(0)
            st = emu.emu_fft_product(s.ctypes.data_as(C.POINTER(C.c_double)), wide.ctypes.data_as(C.POINTER(C.c_uint64)),
                                     center, log_n, q, rc, c.ctypes.data_as(C.POINTER(C.c_uint64)), C.byref(off))
            assert st == 0, (name, st)
            assert np.array_equal(c, ref), name
            assert off.value <= bound, (name, off.value, bound)
            assert emu.emu_fft_layout_ok() == 1
