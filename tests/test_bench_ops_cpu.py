"""The operation counts behind the benchmark's fractions of the device's peak rates."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_square_counts_its_own_transforms():
    """Image matching multiplies a buffer by itself.  At N = 8192 and 4 primes the square takes 2
    forward and 1 inverse transforms per prime for the tensor product, 4 + 2 in the special prime,
    and 3 + 2 per prime for key switching: 38, where two different factors would take 46."""
    import bench

    N, L = 8192, 4
    transforms = 3 * L + (L + 2) + L * (L - 1 + 2)
    assert transforms == 38
    products = 6 * L + 2 * L * (L + 1) + 4 * L
    assert bench.mul_ops_per_square(13, L) == transforms * 8 * (N // 2) * 13 + products * 6 * N
