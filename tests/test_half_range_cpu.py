"""The test by which a step of 64 contraction indices is given to two scaled fp16 numbers per operand (gemm_half.hip), in numpy: what it
lets pass is within the stated part of the sum of |a||x|, and ordinary numbers pass."""
import numpy as np
import pytest

MIN_RUNS, MAX_SMALL, LARGE_RUN, LARGE_ENTRY = (14, 7), (11, 5), 2.0 ** -7, 2.0 ** -9


def _passes(a, x, top, whole):
    """a: a row's step, x: one column of the panel's step, top: the largest of all of that step's columns.  Run = four successive indices."""
    n = 64 if whole else 32
    runs = np.abs(a).reshape(16, 4).max(1)[:n // 4]
    small = int((np.abs(x[:n]) < top * LARGE_ENTRY).sum())
    k = 0 if whole else 1
    return int((runs >= np.abs(a).max() * LARGE_RUN).sum()) >= MIN_RUNS[k] and (small <= MAX_SMALL[k] or not x.any())


def _split(v, top):
    """h and l of numbers under the scale of `top`, in units of that scale."""
    scale = 2.0 ** (14 - np.floor(np.log2(top)))
    h = (v * scale).astype(np.float32).astype(np.float16)
    return h, ((v * scale).astype(np.float32) - h.astype(np.float32)).astype(np.float16), scale


def _error(a, x, top):
    """Of the three products taken, to the sum of |a||x|."""
    ah, al, sa = _split(a, np.abs(a).max())
    xh, xl, sx = _split(x, top)
    ah, al, xh, xl = (v.astype(np.float64) for v in (ah, al, xh, xl))
    exact, scale = a.astype(np.float64) * x, np.abs(a.astype(np.float64) * x).sum()
    return abs(((al * xh + ah * xl + ah * xh) / (sa * sx) - exact).sum()) / scale if scale else 0.0


def _cases(rng):
    """Rows and columns with many numbers that one scale loses, around what the test lets pass."""
    whole = bool(rng.integers(2))
    tiny = lambda shape: rng.choice([-1.0, 1.0], shape) * 2.0 ** -rng.uniform(15.0, 45.0, shape)
    a, x = tiny(64), tiny(64) if rng.integers(2) else rng.choice([-1.0, 1.0], 64)
    n = 16 if whole else 8
    large = 4 * rng.choice(n, rng.integers(n - 4, n + 1), replace=False) + rng.integers(0, 4)
    a[large] = 2.0 ** -rng.uniform(5.0, 8.0)
    a[rng.integers(0, 64)] = 1.0
    x[large] = rng.choice([1.0, 2.0 ** -8, 2.0 ** -9], len(large))
    x[rng.choice(large, min(len(large), rng.integers(0, 13)), replace=False)] = rng.choice([0.0, 1e-12])
    if not whole:
        x[32 + rng.integers(0, 32):] = 0.0
    return a.astype(np.float32), x.astype(np.float32), whole


def test_what_passes_is_accurate():
    rng = np.random.default_rng(7)
    passed = 0
    for _ in range(20000):
        a, x, whole = _cases(rng)
        if not _passes(a, x, 1.0, whole):
            continue
        passed += 1
        assert _error(a, x, 1.0) <= 2.0 ** (-18 if whole else -17)
    assert passed > 1000


@pytest.mark.parametrize("make", [lambda g: g.standard_normal(64), lambda g: g.random(64), lambda g: g.exponential(size=64)])
def test_ordinary_numbers_pass(make):
    rng = np.random.default_rng(8)
    for _ in range(2000):
        a, x = make(rng), rng.standard_normal(64)
        assert _passes(a, x, 4.5, True) and _passes(a, x, 4.5, False)


def test_single_large_number_does_not_pass():
    a, x = np.full(64, 1.37 * 2.0 ** -30, np.float32), np.ones(64, np.float32)
    a[5], x[5] = 1.0, 0.0
    assert not _passes(a, x, 1.0, True) and _error(a, x, 1.0) > 1e-5
