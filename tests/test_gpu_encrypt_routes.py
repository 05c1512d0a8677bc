"""Encryption by each of its kernels -- a pixel split over workgroups, whole ciphertexts through
prime-field and through complex transforms -- against the oracle.  The counts are chosen for a
device of 256 compute units."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#         log N, primes, bits, log scale, width, pixels
ROUTES = [(11, 1, 30, 18, 8, (3, 65)), (12, 1, 36, 28, 8, (3, 1025)),
          (13, 1, 50, 38, 8, (128, 200, 512)), (13, 2, 50, 40, 8, (128, 129, 256, 257)), (13, 4, 50, 40, 8, (171, 256)),
          # every class of primes at every ring, the shortest of the upper class (41 bits) where the
          # quotient of the high piece alone is tightest; the last count takes complex transforms
          (11, 4, 20, 10, 8, (5, 200, 2048)), (11, 4, 40, 30, 8, (5, 200, 2048)), (11, 4, 41, 30, 8, (5, 200, 2048)),
          (11, 4, 50, 38, 8, (5, 200, 2048)), (12, 3, 40, 30, 8, (5, 200, 1024)), (12, 3, 41, 30, 8, (5, 200, 1024)),
          (12, 3, 50, 40, 8, (5, 200, 1024)), (13, 3, 36, 28, 8, (5, 200, 1000)), (13, 2, 40, 30, 8, (5, 200, 300)),
          (13, 2, 41, 30, 8, (5, 200, 300)), (14, 2, 36, 26, 16, (5, 130)), (14, 2, 40, 30, 16, (5, 130)),
          (14, 2, 41, 30, 16, (5, 130)), (13, 1, 36, 26, 8, (8300,))]


@pytest.mark.parametrize("log_n,L,bits,log_scale,width,counts", ROUTES)
def test_encryption_matches_oracle(oracle_mod, log_n, L, bits, log_scale, width, counts):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.set_ntt_width(width)
    ctx.keygen((51, log_n))
    o = oracle_mod.Oracle(log_n, L, bits, log_scale)
    o.keygen((51, log_n))
    rng = np.random.default_rng([log_n, bits])
    for n in counts:
        print("[gpu] encryption N=2^%d %dx%d bits width %d, %d pixels" % (log_n, L, bits, width, n), flush=True)
        px = rng.integers(0, 256, n, dtype=np.uint8)
        px[:3] = (255, 0, 1)[:min(n, 3)]
        got = ctx.encrypt_pixels(torch.from_numpy(px).cuda(), (52, n), first_index=9)
        data = got.data.view(n, -1)
        for i in sorted({0, 1, n // 2, n - 1}):
            ref = o.encrypt_batch(px[i:i + 1], (52, n), first_index=9 + i)
            assert np.array_equal(data[i].cpu().numpy().view(np.uint64), np.asarray(ref).reshape(-1)), (n, i)
        # every ciphertext and value by smaller calls, which take other kernels
        values = ctx.decrypt_pixels(got)
        step = 100 if n <= 1100 else 700
        for a in range(0, n, step):
            part = ctx.encrypt_pixels(torch.from_numpy(px[a:a + step]).cuda(), (52, n), first_index=9 + a)
            assert torch.equal(part.data.view(part.count, -1), data[a:a + step]), (n, a)
            assert torch.equal(ctx.decrypt_pixels(part), values[a:a + step]), (n, a)
        values = values.cpu()
        for i in (0, n - 1):  # sums of N terms of up to 2 x 255 / N and noise: 1e-12 of rounding
            ref = o.decrypt(data[i].cpu().numpy().view(np.uint64).reshape(2, L, -1))
            assert abs(float(values[i]) - ref) < 1e-9, (n, i)
