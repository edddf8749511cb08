"""The quantizer takes range / q_max as a product with the rounded reciprocal, its exact remainder and one correction (two fused multiply-adds). Here
the same steps in exact arithmetic, at every fp32 significand, against the IEEE quotient (scaling by a power of two changes nothing: a range of
fp16 numbers is far from the ends of the exponent range)."""
import numpy as np
import pytest


@pytest.mark.parametrize("q_max", [3, 7, 15])
def test_range_over_q_max_is_the_ieee_quotient(q_max):
    x = np.arange(1 << 23, dtype=np.uint32)
    x = (x | np.uint32(0x3F800000)).view(np.float32)                  # [1, 2)
    inv = np.float32(1.0) / np.float32(q_max)
    q = x * inv                                                       # rounded once
    rest = x.astype(np.float64) - q_max * q.astype(np.float64)        # at most 28 bits: exact, and so is its fp32 image
    assert np.array_equal(rest.astype(np.float32), rest)
    t = rest * np.float64(inv)                                        # 48 bits: exact
    power_of_two = (q.view(np.uint32) & np.uint32(0x7FFFFF)) == 0
    unit = np.spacing(q).astype(np.float64) * np.where((t < 0) & power_of_two, 0.5, 1.0)      # spacing on the side of q that t points to
    step = t / unit                                                   # (a power of two) what the fused operation adds to q, before its rounding
    assert np.abs(step).max() < 2.0 and not (np.abs(np.abs(step) - np.floor(np.abs(step))) == 0.5).any()
    got = (q.astype(np.float64) + np.rint(step) * unit).astype(np.float32)
    assert np.array_equal(got, x / np.float32(q_max))
