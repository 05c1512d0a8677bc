"""The decoded value of a ciphertext does not depend on how many are decrypted by one call: the
kernels for few and for many ciphertexts sum in the order of the context's width."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [8, 16, 32])
@pytest.mark.parametrize("level", [1, 4])
def test_value_is_independent_of_the_call_size(width, level):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2409_03568_amd as P

    n = 17 * torch.cuda.get_device_properties(0).multi_processor_count
    print("[gpu] decode order, width %d, level %d, %d ciphertexts" % (width, level, n), flush=True)
    ctx = P.Context(13, 4, 50, 40)
    ctx.set_ntt_width(width)
    ctx.keygen((31, width))
    cts = ctx.encrypt_pixels(torch.from_numpy((np.arange(n) % 256).astype(np.uint8)).cuda(), (32, width))
    while cts.level > level:
        cts = ctx.rescale(ctx.mul_const(cts, 0.5))
    whole = ctx.decrypt_pixels(cts)
    for first, count in ((0, 1), (1, 7), (100, 200), (7, 300), (300, n // 2)):
        part = ctx.decrypt_pixels(cts[first:first + count])
        assert torch.equal(part, whole[first:first + count]), (first, count)
