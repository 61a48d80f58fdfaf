"""LayerNorm's mean and variance: a float64 product with 1 / d, rounded once to float32, in place of a float32 division.

The quotient of a float32 by an integer d < 2^12 lies on a boundary between two float32 values or at least 2^-37 of itself away from it; the product
is off by 2^-52 of itself at most.  So the two round alike, and where the quotient is below the normal range they do for all that is tried here.
"""
import numpy as np
import pytest


@pytest.mark.parametrize("d", [*range(64, 2049, 64), 4, 12, 100, 1020, 2044])   # widths of the kernels that keep a row in registers
def test_product_in_float64_is_the_float32_quotient(d):
    rng = np.random.default_rng(d)
    bits = np.concatenate([rng.integers(0, 0x7F800000, 400_000), rng.integers(0, 1 << 25, 100_000),      # all finite values; subnormal ones
                           np.arange(3000, dtype=np.float32).view(np.uint32), [0x7F800000, 0x7F7FFFFF, 0, 1, 0x00800000]]).astype(np.uint32)
    s = bits.view(np.float32)
    with np.errstate(all="ignore"):
        got = (s.astype(np.float64) * (1.0 / d)).astype(np.float32)
        np.testing.assert_array_equal(got, s / np.float32(d))
        np.testing.assert_array_equal((-s.astype(np.float64) * (1.0 / d)).astype(np.float32), -s / np.float32(d))
        # multiples of d: the values themselves
        c = np.arange(-4000, 4000, dtype=np.float32)
        np.testing.assert_array_equal(((c * np.float32(d)).astype(np.float64) * (1.0 / d)).astype(np.float32), c)
