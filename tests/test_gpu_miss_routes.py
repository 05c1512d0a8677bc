"""Value-cached encryption through each choice that the device makes by the number of misses: few
misses, about half, and nearly all, on both sides of the lines, against plain encryption of the
missed pixels and the gather of the others by a small call."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RINGS = {11: (3, 30, 20), 12: (3, 36, 30), 13: (2, 50, 40), 14: (1, 50, 38)}


@pytest.mark.parametrize("log_n", [11, 12, 13, 14])
@pytest.mark.parametrize("n", [200, 1100, 1500])
@pytest.mark.parametrize("missing", [0.0, 0.02, 0.3, 0.34, 0.5, 0.95, 1.0])
def test_every_share_of_misses(log_n, n, missing):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    print("[gpu] misses N=2^%d, %d pixels, %.2f missing" % (log_n, n, missing), flush=True)
    ctx = P.Context(log_n, *RINGS[log_n])
    ctx.keygen((61, log_n))
    # the cache holds value 7; m of the pixels have others
    m = int(round(missing * n))
    px = np.full(n, 7, dtype=np.uint8)
    at = np.random.default_rng([log_n, n, m]).permutation(n)[:m]
    px[at] = 20 + np.arange(m) % 200
    scan = torch.full((8,), 7, dtype=torch.uint8, device="cuda")
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=1, zero_pool=4, scan_px=scan, seed=(62, log_n))
    dev = torch.from_numpy(px).cuda()
    got = ctx.encrypt_cached(cache, dev, (63, n), 3).data.view(n, -1)
    plain = ctx.encrypt_pixels(dev, (63, n), 3).data.view(n, -1)
    torch.cuda.synchronize()
    miss = torch.from_numpy(px != 7).cuda()
    assert torch.equal(got[miss], plain[miss])
    # hits, piece by piece: calls of at most 64 pixels
    for a in range(0, n, 64):
        part = ctx.encrypt_cached(cache, dev[a:a + 64].contiguous(), (63, n), 3 + a).data.view(min(64, n - a), -1)
        assert torch.equal(got[a:a + 64], part), a
    cache.close()
    ctx.close()


@pytest.mark.parametrize("log_n", [11, 12, 13, 14])
@pytest.mark.parametrize("n", [100, 300, 600, 3100])
@pytest.mark.parametrize("missing", [0.02, 0.5, 1.0])
def test_without_allocation(log_n, n, missing):
    """The entry point without allocations encrypts the misses after the gather, by lines of its own;
    its ciphertexts equal those of the one that does both at once."""
    import ctypes as C

    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    print("[gpu] misses without allocation N=2^%d, %d pixels, %.2f missing" % (log_n, n, missing), flush=True)
    ctx = P.Context(log_n, *RINGS[log_n])
    ctx.keygen((64, log_n))
    m = int(round(missing * n))
    px = np.full(n, 7, dtype=np.uint8)
    px[np.random.default_rng([log_n, n, m]).permutation(n)[:m]] = 20
    scan = torch.full((8,), 7, dtype=torch.uint8, device="cuda")
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=1, zero_pool=4, scan_px=scan, seed=(65, log_n))
    dev, out = torch.from_numpy(px).cuda(), ctx.empty(n)
    b = out.out_batch()
    rc = P.lib().ckks_encrypt_cached_noalloc(ctx.handle, cache.handle, C.c_void_p(dev.data_ptr()), n, P._seed((66, n)), 3,
                                              C.byref(b), P._stream(None))
    assert rc == 0, P.ckks_last_error()
    want = ctx.encrypt_cached(cache, dev, (66, n), 3)
    torch.cuda.synchronize()
    assert torch.equal(out.data, want.data)
    cache.close()
    ctx.close()


@pytest.mark.parametrize("primes", [3, 4, 8])
@pytest.mark.parametrize("n", [129, 171, 240, 241, 256, 257, 512, 513, 1537])
@pytest.mark.parametrize("missing", [0.0, 0.05, 0.6, 1.0])
def test_short_lists(primes, n, missing):
    """Lists of up to some pixels per CU, whose kernel goes by the primes too: on either stream the
    ciphertexts of the misses are those of plain calls of at most 64 pixels."""
    import ctypes as C

    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    print("[gpu] short list %d primes, %d pixels, %.2f missing" % (primes, n, missing), flush=True)
    ctx = P.Context(13, primes, 50, 40)
    ctx.keygen((67, primes))
    m = int(round(missing * n))
    px = np.full(n, 7, dtype=np.uint8)
    px[np.random.default_rng([primes, n, m]).permutation(n)[:m]] = 20
    scan = torch.full((8,), 7, dtype=torch.uint8, device="cuda")
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=1, zero_pool=4, scan_px=scan, seed=(68, primes))
    dev, out = torch.from_numpy(px).cuda(), ctx.empty(n)
    b = out.out_batch()
    rc = P.lib().ckks_encrypt_cached_noalloc(ctx.handle, cache.handle, C.c_void_p(dev.data_ptr()), n, P._seed((69, n)), 3,
                                              C.byref(b), P._stream(None))
    assert rc == 0, P.ckks_last_error()
    beside = ctx.encrypt_cached(cache, dev, (69, n), 3)
    torch.cuda.synchronize()
    assert torch.equal(out.data, beside.data)
    for a in range(0, n, 64):
        part = ctx.encrypt_pixels(dev[a:a + 64].contiguous(), (69, n), 3 + a).data.view(min(64, n - a), -1)
        miss = torch.from_numpy(px[a:a + 64] != 7).cuda()
        assert torch.equal(beside.data.view(n, -1)[a:a + 64][miss], part[miss]), a
    cache.close()
    ctx.close()


@pytest.mark.parametrize("n", [1535, 1537, 4097])
@pytest.mark.parametrize("log_n", [11, 12])
@pytest.mark.parametrize("missing", [0.02, 1.0])
def test_eight_primes(log_n, n, missing):
    """Eight primes at the smaller rings, counted after the gather from a length of their own on."""
    import ctypes as C

    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    print("[gpu] misses of 8 primes N=2^%d, %d pixels, %.2f missing" % (log_n, n, missing), flush=True)
    ctx = P.Context(log_n, 8, 36 if log_n == 12 else 30, 30 if log_n == 12 else 20)
    ctx.keygen((70, log_n))
    m = int(round(missing * n))
    px = np.full(n, 7, dtype=np.uint8)
    px[np.random.default_rng([log_n, n, m]).permutation(n)[:m]] = 20
    scan = torch.full((8,), 7, dtype=torch.uint8, device="cuda")
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=1, zero_pool=4, scan_px=scan, seed=(71, log_n))
    dev, out = torch.from_numpy(px).cuda(), ctx.empty(n)
    b = out.out_batch()
    rc = P.lib().ckks_encrypt_cached_noalloc(ctx.handle, cache.handle, C.c_void_p(dev.data_ptr()), n, P._seed((72, n)), 3,
                                              C.byref(b), P._stream(None))
    assert rc == 0, P.ckks_last_error()
    beside = ctx.encrypt_cached(cache, dev, (72, n), 3)
    plain = ctx.encrypt_pixels(dev, (72, n), 3)
    torch.cuda.synchronize()
    assert torch.equal(out.data, beside.data)
    miss = torch.from_numpy(px != 7).cuda()
    assert torch.equal(beside.data.view(n, -1)[miss], plain.data.view(n, -1)[miss])
    cache.close()
    ctx.close()
