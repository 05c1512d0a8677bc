"""Encryption by each of its kernels -- a pixel split over workgroups, whole ciphertexts through
prime-field and through complex transforms -- against the oracle.  The counts are chosen for a
device of 256 compute units."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#         log N, primes, bits, log scale, width, pixels
ROUTES = [(11, 1, 30, 18, 8, (3, 65)), (12, 1, 36, 28, 8, (3, 1025)),
          (13, 1, 50, 38, 8, (128, 200, 512)), (13, 2, 50, 40, 8, (128, 129, 256, 257)), (13, 4, 50, 40, 8, (171, 256))]


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
        # every ciphertext, through its decryption: fresh noise of about 2^8 per coefficient
        off = float((ctx.decrypt_pixels(got).cpu() - torch.from_numpy(px).double()).abs().max())
        assert off < 8 * 2.0**8 * np.sqrt(2.0**log_n / 2) / 2.0**log_scale, (n, off)
