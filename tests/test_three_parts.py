"""The cut of an fp32 value into three bfloat16 parts that the dense products of any shape rest on, restated in numpy:
parts rounded to nearest add up to the value exactly, and the products that are left out stay below the rounding of
one fp32 product, in either direction."""
import numpy as np


def _bf16(x):
    """nearest bfloat16, ties to even, as fp32"""
    b = np.asarray(x, np.float32).view(np.uint32).astype(np.uint64)
    return ((b + 0x7FFF + ((b >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def _parts(x):
    hi = _bf16(x)
    mid = _bf16(x - hi)
    return hi, mid, (x - hi) - mid


def _values(rng, n):
    b = rng.integers(0, 1 << 24, n, dtype=np.uint32) | rng.integers(60, 195, n, dtype=np.uint32) << 23 | rng.integers(0, 2, n, dtype=np.uint32) << 31
    edge = np.array([0.0, 1.0, -1.0, 1.0 + 2.0 ** -23, 2.0 - 2.0 ** -23, 1.0 + 2.0 ** -8, 1.0 + 2.0 ** -8 + 2.0 ** -17], np.float32)
    return np.concatenate([b.view(np.float32), np.array([0x3F80FFFF, 0x3F807FFF, 0x3F808000, 0x3F817F7F], np.uint32).view(np.float32), edge])


def test_three_parts_are_exact_bfloat16_values():
    x = _values(np.random.default_rng(1), 200000)
    hi, mid, lo = _parts(x)
    assert np.array_equal(_bf16(lo), lo)                                # the third part needs no rounding
    assert np.array_equal(hi.astype(np.float64) + mid + lo, x.astype(np.float64))
    assert np.all(np.abs(mid) <= 2.0 ** -8 * np.abs(x)) and np.all(np.abs(lo) <= 2.0 ** -17 * np.abs(x))


def test_products_left_out_are_below_one_rounding_and_have_no_direction():
    rng = np.random.default_rng(2)
    x, y = _values(rng, 200000), _values(rng, 200000)
    (_, xm, xl), (_, ym, yl) = _parts(x), _parts(y)
    xm, xl, ym, yl = (v.astype(np.float64) for v in (xm, xl, ym, yl))
    whole = np.abs(x.astype(np.float64) * y)
    left_out = xm * yl + xl * ym + xl * yl
    assert np.all(np.abs(left_out) <= 2.0 ** -24 * (1.0 + 2.0 ** -9) * whole)
    share = left_out[whole > 0] / whole[whole > 0] * (np.sign(x) * np.sign(y))[whole > 0] * 2.0 ** 24
    assert abs(share.mean()) < 0.002 and share.std() < 0.2               # (truncated parts: mean 0.63)
