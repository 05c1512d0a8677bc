"""Encryption and decryption by each of their kernels.  Which one runs depends on the ring degree
and the number of ciphertexts: a pixel split over workgroups, whole ciphertexts through
prime-field transforms, or whole ciphertexts through complex transforms.  The counts here lie on
both sides of every line, for a device of 256 compute units, and the ciphertexts of any count
equal those of the oracle and of one call for all pixels, the decoded values the pixels."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

#        log_n, L, prime bits, log scale, counts
ROUTES = [(11, 3, 30, 20, (1, 63, 64, 65, 8191, 8192)), (12, 3, 36, 30, (1, 43, 128, 129, 511, 512)),
          (13, 4, 50, 40, (1, 85, 128, 129, 256, 257)), (14, 2, 50, 40, (1, 85, 128, 129))]


@pytest.fixture(scope="module")
def P():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    P.lib()
    return P


@pytest.mark.parametrize("log_n,L,bits,log_scale,counts", ROUTES)
def test_encryption_routes(P, oracle_mod, log_n, L, bits, log_scale, counts):
    import torch

    most = max(counts)
    px = torch.from_numpy(np.random.default_rng(log_n).integers(0, 256, most, dtype=np.uint8)).cuda()
    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.keygen((21, log_n))
    o = oracle_mod.Oracle(log_n, L, bits, log_scale)
    o.keygen((21, log_n))
    every = ctx.encrypt_pixels(px, (22, log_n), first_index=7)
    whole = every.data.view(most, -1)
    for i in (0, most - 1):
        ref = o.encrypt_batch(px[i:i + 1].cpu().numpy(), (22, log_n), first_index=7 + i)
        assert np.array_equal(whole[i].cpu().numpy().view(np.uint64), np.asarray(ref).reshape(-1)), i
    for n in counts:
        print("[gpu] routes N=2^%d n=%d" % (log_n, n), flush=True)
        part = ctx.encrypt_pixels(px[most - n:].contiguous(), (22, log_n), first_index=7 + most - n)
        assert torch.equal(part.data.view(n, -1), whole[most - n:]), n
        # encryption noise: |v e + e0 + e1 s| in slot 0 stays far below 2^-8 of a grey level
        dec = ctx.decrypt_pixels(part)
        assert float((dec - px[most - n:].double()).abs().max()) < 0.25, n
        del part


@pytest.mark.parametrize("log_n,L,bits,log_scale", [r[:4] for r in ROUTES[:3]])
@pytest.mark.parametrize("n", [3, 300])
def test_miss_lists_and_batches(P, log_n, L, bits, log_scale, n):
    """A cache's misses through the list forms of the kernels: equal to plain encryptions of the
    same pixels; and a batch through a ring smaller than its misses decodes as one that keeps
    every ciphertext."""
    import torch

    px = torch.from_numpy((np.arange(n) % 5).astype(np.uint8)).cuda()
    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.keygen((23, log_n))
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_TOPK, topk=2, zero_pool=4, scan_px=px, seed=(24, log_n))
    plain = ctx.encrypt_pixels(px, (25, log_n)).data.view(n, -1)
    got = ctx.encrypt_cached(cache, px, (25, log_n)).data.view(n, -1)
    same = (plain == got).all(dim=1).cpu().numpy()
    hit = {int(v) for v in px.cpu().numpy()[~same]}
    assert len(hit) == 2 and same.sum() == sum(int(v) not in hit for v in px.cpu().numpy())
    seg, b = np.array([1, n], dtype=np.uint64), np.array([2.0, -3.0])
    out = []
    for chunk, keep in ((max(1, n // 7), False), (n, True)):
        plan = P.BatchPlan(ctx, cache, chunk, False)
        cts = ctx.empty(n) if keep else None
        out.append(plan.run(px, seg, b, (25, log_n), cts_out=cts) if keep else plan.run(px, seg, b, (25, log_n)))
        torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
    want = px.double() + torch.tensor([2.0] + [-3.0] * (n - 1), dtype=torch.float64, device="cuda")
    assert float((out[0] - want).abs().max()) < 0.5


@pytest.mark.parametrize("log_n,L,bits,log_scale", [r[:4] for r in ROUTES])
@pytest.mark.parametrize("level", [1, 2, 0])
def test_square_is_the_product(P, log_n, L, bits, log_scale, level):
    """The product of a buffer with itself takes half the forward transforms; it equals the product
    with a copy, also where the result replaces the factor."""
    import torch

    px = torch.arange(0, 255, 51, dtype=torch.uint8, device="cuda")
    ctx = P.Context(log_n, L, bits, log_scale)
    ctx.keygen((26, log_n))
    ctx.relin_keygen((27, log_n))
    a = ctx.encrypt_pixels(px, (28, log_n))
    while level and a.level > level:
        a = ctx.rescale(a)
    b = P.Ciphertexts(a.data.clone(), a.level, a.scale)
    want = ctx.mul(a, b).data.clone()
    assert torch.equal(ctx.mul(a, a).data, want)
    assert torch.equal(ctx.mul(b, b, out=b).data, want)
