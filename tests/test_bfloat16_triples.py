"""The arithmetic of the wide kernels, emulated on the CPU: a 32-bit float is the exact sum of three bfloat16, the six
partial products that the kernels form are within the tolerance that their tests allow a single product, and
leaving out any one of the six is not."""
import itertools

import numpy as np
import pytest

KEPT = [(0, 0), (0, 1), (1, 0), (1, 1), (0, 2), (2, 0)]


def to_bfloat16(v):
    """Nearest, ties to even, of finite 32-bit floats that do not overflow."""
    u = v.astype(np.float32).view(np.uint32)
    return ((u + 0x7FFF + (u >> 16 & 1)) & np.uint32(0xFFFF0000)).view(np.float32)


def triple(v):
    a = to_bfloat16(v)
    b = to_bfloat16(v - a)
    return np.stack([a, b, to_bfloat16(v - a - b)]).astype(np.float64)


def floats(seed, n):
    rng = np.random.default_rng(seed)
    v = (rng.uniform(1, 2, n) * np.where(rng.random(n) < 0.5, -1, 1)).astype(np.float32)
    edges = np.array([1.0, 1 + 2.0 ** -23, 2 - 2.0 ** -23, 1 + 2.0 ** -8, 1 + 2.0 ** -8 + 2.0 ** -23, 1 + 2.0 ** -9, 1 + 2.0 ** -16, 1 + 2.0 ** -17,
                      1.99609375, 1.998046875 - 2.0 ** -23], np.float32)
    v[:len(edges)] = edges
    return v


@pytest.mark.parametrize("exponent", [-100, -60, 0, 90, 126])
def test_triples_are_exact(exponent):
    v = floats(9300, 200000) * np.float32(2.0) ** exponent
    assert np.array_equal(triple(v).sum(0), v.astype(np.float64))


def test_six_products_and_no_fewer():
    w, x = floats(9301, 100000), floats(9302, 100000)
    wt, xt, exact = triple(w), triple(x), w.astype(np.float64) * x

    def error(pairs):
        return np.abs(sum(wt[i] * xt[j] for i, j in pairs) - exact) / np.abs(exact)

    # b is at most 2^-8 and c 2^-17 of the operand, so the two largest of what is left out are at most 2^-25 each
    assert error(KEPT).max() <= 2.0 ** -24 * (1 + 2.0 ** -9)
    assert np.sqrt((error(KEPT) ** 2).mean()) <= 2.0 ** -27
    for left_out in range(6):
        assert error([p for k, p in enumerate(KEPT) if k != left_out]).max() > 2.25 * 2.0 ** -24    # the tests' tolerance
    assert error(itertools.product(range(3), range(3))).max() == 0
