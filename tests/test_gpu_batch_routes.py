"""Batches through each of their routes -- one persistent launch with or without the misses, and
misses apart through a ring -- against the unbatched calls: ciphertexts and decoded values bit for
bit, at every width."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

RINGS = {11: (3, 30, 20), 12: (3, 36, 30), 13: (4, 50, 40), 14: (2, 50, 40)}


#        log N, width, kind, pixels, chunk
@pytest.mark.parametrize("log_n,width,kind,n,chunk", [
    (11, 8, "topk", 300, 7), (11, 16, "topk", 300, 512), (11, 32, "plain", 200, 64), (11, 8, "plain", 300, 300),
    (12, 8, "topk", 300, 64), (12, 32, "topk", 150, 9), (12, 16, "plain", 400, 256), (12, 8, "plain", 200, 64),
    (13, 8, "topk", 300, 64), (13, 16, "topk", 300, 512), (13, 8, "topk", 2100, 600), (13, 32, "plain", 300, 256),
    (13, 16, "plain", 700, 512), (14, 16, "topk", 40, 7), (14, 32, "plain", 1030, 1), (14, 16, "topk", 1030, 1)])
def test_routes_match_unbatched(log_n, width, kind, n, chunk):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    L, bits, log_scale = RINGS[log_n]
    print("[gpu] batch route N=2^%d width %d %s, %d pixels, chunk %d" % (log_n, width, kind, n, chunk), flush=True)
    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.set_ntt_width(width)
    ctx.keygen((41, log_n))
    px = torch.from_numpy(np.random.default_rng(n).integers(0, 12, n, dtype=np.uint8)).cuda()
    cache = None
    if kind == "topk":
        cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=7, zero_pool=4, scan_px=px, seed=(42, log_n))
    seg, b = np.array([n // 3, n], dtype=np.uint64), np.array([3.0, -7.0])
    per_ct = torch.from_numpy(np.repeat(b, [n // 3, n - n // 3])).cuda()
    want = ctx.encrypt_cached(cache, px, (43, n), 5) if cache else ctx.encrypt_pixels(px, (43, n), 5)
    ctx.add_const(want, per_ct=per_ct)
    decoded = ctx.decrypt_pixels(want)
    plan = P.BatchPlan(ctx, cache, chunk, False)
    cts = ctx.empty(n)
    kept = plan.run(px, seg, b, (43, n), 5, cts_out=cts)
    through_ring = plan.run(px, seg, b, (43, n), 5)
    torch.cuda.synchronize()
    assert torch.equal(cts.data, want.data)
    assert torch.equal(kept, decoded)
    assert torch.equal(through_ring, decoded)
    plan.close()


@pytest.mark.parametrize("missing", [0, 1, 127, 128, 129, 900, 1700])
@pytest.mark.parametrize("keep", [False, True])
def test_misses_counted_on_the_device(missing, keep):
    """At N = 8192 the device lets the misses' own launches run from half a wave of misses on (128 on
    256 compute units), and the persistent launch take them below that."""
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    n, ring = 1700, 600
    print("[gpu] counted misses %d of %d, ring %d, kept %s" % (missing, n, ring, keep), flush=True)
    ctx = P.Context(13, 2, 50, 40)
    ctx.keygen((44, 13))
    px = np.full(n, 9, dtype=np.uint8)
    px[np.random.default_rng(missing).permutation(n)[:missing]] = 200
    dev = torch.from_numpy(px).cuda()
    scan = torch.full((4,), 9, dtype=torch.uint8, device="cuda")
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=1, zero_pool=4, scan_px=scan, seed=(45, 13))
    want = ctx.encrypt_cached(cache, dev, (46, missing))
    ctx.add_const(want, 4.0)
    decoded = ctx.decrypt_pixels(want)
    plan = P.BatchPlan(ctx, cache, ring, True)
    cts = ctx.empty(n) if keep else None
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    for rep in range(4):  # eager, then replays of the captured launches, with other work between
        out.fill_(-1.0)
        if keep:
            cts.data.zero_()
            plan.run(dev, np.array([n], dtype=np.uint64), np.array([4.0]), (46, missing), out=out, cts_out=cts)
        else:
            plan.run(dev, np.array([n], dtype=np.uint64), np.array([4.0]), (46, missing), out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, decoded), rep
        if keep:
            assert torch.equal(cts.data, want.data), rep
        ctx.encrypt_pixels(dev[:300].contiguous(), (47, rep))
        torch.cuda.synchronize()
    plan.close()
    cache.close()
