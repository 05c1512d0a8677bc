"""The prime-field encryption kernel at every width, by counts that reach it: plain pixels, miss
lists and fused brightness, against the oracle.  (Smaller calls are split over workgroups by a kernel
that has no width.)  The counts are chosen for a device of 256 compute units."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#        log N, primes, bits, log scale, pixels
RINGS = [(11, 3, 30, 20, 300), (12, 3, 36, 30, 300), (13, 4, 50, 40, 200)]
WIDTHS = [8, 16, 32]


def _ctx(ring, width):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    log_n, L, bits, log_scale, n = ring
    print("[gpu] width route N=2^%d width %d, %d pixels" % (log_n, width, n), flush=True)
    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.set_ntt_width(width)
    ctx.keygen((71, log_n))
    px = np.random.default_rng(log_n).integers(0, 256, n, dtype=np.uint8)
    return P, ctx, px, torch.from_numpy(px).cuda()


def _oracle(oracle_mod, ring):
    o = oracle_mod.Oracle(*ring[:4])
    o.keygen((71, ring[0]))
    return o


def _u64(t):
    return t.cpu().numpy().view(np.uint64)


@pytest.mark.parametrize("ring", RINGS)
@pytest.mark.parametrize("width", WIDTHS)
def test_pixels(oracle_mod, ring, width):
    P, ctx, px, dev = _ctx(ring, width)
    o, n = _oracle(oracle_mod, ring), px.size
    got = _u64(ctx.encrypt_pixels(dev, (72, n), first_index=4).data.view(n, -1))
    for i in (0, 1, n // 2, n - 1):
        assert np.array_equal(got[i], np.asarray(o.encrypt_batch(px[i:i + 1], (72, n), first_index=4 + i)).reshape(-1)), i


@pytest.mark.parametrize("ring", RINGS)
@pytest.mark.parametrize("width", WIDTHS)
def test_miss_lists(oracle_mod, ring, width):
    P, ctx, px, dev = _ctx(ring, width)
    o, n = _oracle(oracle_mod, ring), px.size
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=8, zero_pool=4, scan_px=dev, seed=(73, ring[0]))
    kept = set(int(v) for v in o.topk(o.histogram(px), 8))
    got = _u64(ctx.encrypt_cached(cache, dev, (74, n), first_index=6).data.view(n, -1))
    misses = [i for i in range(n) if int(px[i]) not in kept]
    assert len(misses) > n // 2
    for i in misses[:2] + misses[len(misses) // 2:][:1] + misses[-1:]:
        assert np.array_equal(got[i], np.asarray(o.encrypt_batch(px[i:i + 1], (74, n), first_index=6 + i)).reshape(-1)), i


@pytest.mark.parametrize("ring", RINGS)
@pytest.mark.parametrize("width", WIDTHS)
def test_brightness(oracle_mod, ring, width):
    P, ctx, px, dev = _ctx(ring, width)
    o, n = _oracle(oracle_mod, ring), px.size
    plan = P.BatchPlan(ctx, None, n)
    cts = ctx.empty(n)
    value = plan.run(dev, np.array([n // 2, n], dtype=np.uint64), np.array([5.0, -9.0]), (75, n), 8, cts_out=cts).cpu().numpy()
    got = _u64(cts.data.view(n, -1))
    for i in (0, n // 2 - 1, n // 2, n - 1):
        b = 5.0 if i < n // 2 else -9.0
        ref = o.add_const(o.encrypt_batch(px[i:i + 1], (75, n), first_index=8 + i)[0], b)
        assert np.array_equal(got[i], np.asarray(ref).reshape(-1)), i
        assert abs(value[i] - o.decrypt(ref)) < 1e-9, i
    plan.close()
