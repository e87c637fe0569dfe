"""The bound that decides whether a split product may be kept, in NumPy: fp16 halves of scaled fp32
values, x = h + 2^-11 l, over the whole range that the scale admits, against float64."""
import numpy as np
import pytest


def _split(x):
    h = x.astype(np.float16)
    r = (x.astype(np.float64) - h.astype(np.float64)) * 2048.0
    return h.astype(np.float64), r.astype(np.float16).astype(np.float64)


def _low(x):
    return np.maximum(0.0, 1.0 - 8192.0 * np.abs(x.astype(np.float64)))


def _values(rng, shape, lo, hi):
    return np.ldexp(rng.uniform(1.0, 2.0, shape) * rng.choice([-1.0, 1.0], shape),
                    rng.integers(lo, hi, shape)).astype(np.float32)


@pytest.mark.parametrize("lo,hi", [(-60, -25), (-26, -12), (-15, 0), (0, 15)])
def test_one_value(lo, hi):
    x = _values(np.random.default_rng(hi - lo), 200_000, lo, hi)
    h, l = _split(x)
    err = np.abs(x.astype(np.float64) - h - l / 2048.0)
    assert (err <= 2.0 ** -23 * np.abs(x) + 2.0 ** -36 * _low(x)).all()


@pytest.mark.parametrize("lo_a,lo_b", [(-40, -40), (-20, 0), (0, -30), (-13, -13)])
def test_one_product_sum(lo_a, lo_b):
    rng = np.random.default_rng(-lo_a * 50 - lo_b)
    A, B = _values(rng, (64, 48), lo_a, 8), _values(rng, (48, 64), lo_b, 8)
    A[:, 0], B[0] = 1.5, 0.0                      # the value that sets the scale meets a zero
    (ha, la), (hb, lb) = _split(A), _split(B)
    C = ha @ hb + (ha @ lb + la @ hb) / 2048.0
    a, b = A.astype(np.float64), B.astype(np.float64)
    low_a, top_a = _low(A).sum(1)[:, None], np.abs(a).max(1)[:, None]
    low_b, top_b = _low(B).sum(0)[None, :], np.abs(b).max(0)[None, :]
    bound = 2.0 ** -21 * (np.abs(a) @ np.abs(b)) + 2.0 ** -35 * (low_a * top_b + low_b * top_a)
    assert (np.abs(C - a @ b) <= bound).all()
    # the counted weights are the fp16 bits below 2^-13, in 2048ths
    bits = np.ascontiguousarray(np.abs(A.astype(np.float16))).view(np.uint16).astype(np.int64)
    assert np.abs(np.maximum(0, 0x800 - bits) / 2048.0 - _low(A)).max() <= 2.0 ** -11
