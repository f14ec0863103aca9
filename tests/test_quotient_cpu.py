"""The selection's cell coordinates take x / g as trunc((x + 1/2) * (1 / g)) in float32
for 0 <= x <= 2^20: the same arithmetic in NumPy against integer division, every x for
small and power-of-two divisors and a sample of the others, multiples and their
neighbours included."""
import numpy as np

LIMIT = 1 << 20


def quotient(x, g):
    inv = np.float32(1.0) / np.float32(g)
    return ((x.astype(np.float32) + np.float32(0.5)) * inv).astype(np.int64)


def test_every_value_for_grid_sides():
    x = np.arange(LIMIT + 1, dtype=np.int64)
    for g in list(range(1, 130)) + [200, 255, 257, 1000, 1023, 1024, 1025]:
        np.testing.assert_array_equal(quotient(x, g), x // g)


def test_multiples_and_neighbours_for_any_divisor():
    rng = np.random.default_rng(0)
    for g in np.concatenate([rng.integers(130, LIMIT, 400), [LIMIT - 1, LIMIT, LIMIT // 2 + 1]]):
        m = np.arange(0, LIMIT + 1, int(g), dtype=np.int64)
        x = np.unique(np.clip(np.concatenate([m - 1, m, m + 1, [LIMIT]]), 0, LIMIT))
        np.testing.assert_array_equal(quotient(x, int(g)), x // int(g))
