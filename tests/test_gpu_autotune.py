"""The autotuner chooses widths only from timings of kernels that have one, and leaves the tuned
context's results unchanged."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _ctx(*ring, width=None):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    ctx = P.Context(*ring)
    if width:
        ctx.set_ntt_width(width)
    ctx.keygen((81, ring[0]))
    return P, ctx


@pytest.mark.parametrize("ring,trial", [((14, 2, 50, 40), 64), ((12, 3, 36, 30), 100), ((13, 4, 50, 40), 60)])
@pytest.mark.parametrize("width", [16, 32])
def test_no_width_from_kernels_without_one(ring, trial, width):
    """N = 16384 has no prime-field encryption kernel, and the trials at the other rings are small
    enough to be split over workgroups: encryption's width stays what it was."""
    print("[gpu] autotune N=2^%d, %d trials, width %d" % (ring[0], trial, width), flush=True)
    P, ctx = _ctx(*ring, width=width)
    rep = ctx.autotune(trial)
    assert rep["encrypt_width"] == width and ctx.ntt_width() == width
    assert all(math.isinf(v) for v in rep["encrypt_ms"].values())
    assert all(math.isfinite(v) and v > 0 for w, v in rep["decrypt_ms"].items() if (1 << ring[0]) // w <= 1024)


@pytest.mark.parametrize("ring,trial", [((11, 3, 30, 20), 600), ((12, 3, 36, 30), 600), ((13, 4, 50, 40), 600)])
def test_tuned_context_keeps_results(ring, trial):
    import torch

    print("[gpu] autotune N=2^%d, %d trials, results" % (ring[0], trial), flush=True)
    P, ctx = _ctx(*ring)
    ctx.relin_keygen((82, ring[0]))
    px = torch.from_numpy(np.random.default_rng(3).integers(0, 256, 300, dtype=np.uint8)).cuda()
    cache = ctx.cache_build(P.CKKS_CACHE_VALUE_FULL, zero_pool=4, seed=(83, ring[0]))
    plan = P.BatchPlan(ctx, cache, 128)

    def results():
        a, b = ctx.encrypt_pixels(px, (84, 1)), ctx.encrypt_cached(cache, px, (84, 2))
        m = ctx.mul(a, b)
        v = plan.run(px, np.array([300], dtype=np.uint64), np.array([1.0]), (84, 3))
        torch.cuda.synchronize()
        return a.data, b.data, m.data, v, ctx.decrypt_pixels(m)

    before = results()
    rep = ctx.autotune(trial)
    assert all(math.isfinite(v) and v > 0 for k in ("encrypt_ms", "decrypt_ms", "mul_ms") for v in rep[k].values())
    after = results()
    for x, y in zip(before[:3], after[:3]):
        assert torch.equal(x, y)
    # decoded sums follow the width's order: a few units in the last place
    for x, y in zip(before[3:], after[3:]):
        assert float((x - y).abs().max()) <= 1e-9 * max(1.0, float(x.abs().max()))
    plan.close()
    cache.close()
