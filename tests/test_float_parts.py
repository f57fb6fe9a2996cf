"""The three bf16 parts that the float kernels contract a value in (csrc/igemm_stage_kernel.hpp, split3 and store_filter_parts),
emulated on the CPU: exact over the whole range of floats, and the bound that the kernels' header gives for the products left out."""
import numpy as np

SCALE = np.float32(2.0 ** 24)


def bf16(v):
    """v rounded to bf16 (nearest, ties to even), as a float."""
    bits = v.view(np.uint32)
    return ((bits + np.uint32(0x7fff) + ((bits >> np.uint32(16)) & np.uint32(1))) & np.uint32(0xffff0000)).view(np.float32)


def parts(x):
    v = x * SCALE
    p1 = bf16(v)
    r = v - p1
    p2 = bf16(r)
    p3 = r - p2
    return v, p1, p2, p3


def test_every_significand_splits_exactly_and_the_rest_is_bounded():
    x = (np.arange(1 << 23, dtype=np.uint32) | np.uint32(0x3f800000)).view(np.float32)       # [1, 2)
    v, p1, p2, p3 = parts(x)
    assert np.array_equal(bf16(p3), p3)
    assert np.array_equal(p1.astype(np.float64) + p2 + p3, v.astype(np.float64))
    second, third = float(np.max(np.abs(p2 / v))), float(np.max(np.abs(p3 / v)))
    assert second <= 2.0 ** -8 and third <= 2.0 ** -17
    left_out = 2 * second * third + third * third                   # x2 w3 + x3 w2 + x3 w3, over |x w|
    assert left_out <= 2.0 ** -24 * (1 + 2.0 ** -10)


def test_subnormal_and_smallest_floats_have_normal_parts():
    rng = np.random.default_rng(5)
    bits = np.concatenate([np.arange(1, 4096, dtype=np.uint32), rng.integers(1, 0x08000000, 1 << 20, dtype=np.uint32),
                           np.uint32([0x007fffff, 0x00800000, 0x00ffffff])])                  # up to 2^-111
    x = bits.view(np.float32)
    v, p1, p2, p3 = parts(x)
    assert np.array_equal(v.astype(np.float64), x.astype(np.float64) * 2.0 ** 24)
    assert np.array_equal(p1.astype(np.float64) + p2 + p3, v.astype(np.float64))
    for p in (p1, p2, p3):
        assert np.array_equal(bf16(p), p)
        assert np.all((p == 0) | (np.abs(p) >= 2.0 ** -126))
