"""The products of wide fp32 panels over long contractions, whose operands are split into two scaled fp16 numbers: elementwise error
against fp64 at the edges of their tiles, and numbers of every range, which one scale for 64 of them does not hold."""
import pytest
import torch

import paper_1706_07191_amd as B
from tests.gpu_util import need_gpu
from tests.test_gpu_split import _bound, _inputs
from tests.test_gpu_split import test_split_products_not_finite_in_every_part_of_a_plan as _not_finite

pytestmark = pytest.mark.gpu

SHAPES = [  # rows, n, l, elements between A's rows beyond n, offset of A's base; one product or both are of this kind
    (257, 16411, 33, 0, 0),      # one row more than a tile, last step 27 indices, unaligned rows
    (16449, 258, 48, 0, 0),      # A^T Q: last step one index
    (20003, 14016, 17, 0, 0),    # narrowest panel
    (16385, 16390, 80, 0, 0),    # both products, whole steps and one index over
    (16384, 300, 144, 2, 1),     # nine tiles in one column of waves, padded rows, odd base
    (300, 16500, 145, 0, 3),     # ten
    (300, 16500, 161, 0, 0),     # eleven: two columns of waves
    (16500, 301, 208, 0, 0),     # thirteen: seven units of the panel a thread, in two rounds of four
    (400, 16390, 272, 0, 0),     # seventeen
    (16390, 400, 273, 0, 0),     # two column groups
    (300, 20000, 336, 0, 0),     # groups of eleven and ten tiles
    (17000, 300, 512, 0, 0),     # the largest sketch width, two tiles a wave in the packing
    (70000, 1500, 110, 0, 0),    # more row tiles than workgroups: whole contractions and a cut leftover round
]


def _kinds(A, l):
    """Which of the two products are of this kind."""
    rows, n = A.shape
    kinds = [w for w in (0, 1) if B.brsvd_gemm_is_split(w, rows, n, l, A.stride(0), A.data_ptr()) and B.brsvd_gemm_split_parts(w, rows, n, l) == 2]
    assert kinds
    return kinds


def _check_one(w, A, X, Q, bound):
    a, x = (A, X) if w == 0 else (A.T.contiguous(), Q)
    got = B.brsvd_gemm_an(A, X) if w == 0 else B.brsvd_gemm_at(A, Q)
    err = (got.double() - a.double() @ x.double()).abs()
    assert bool((err <= bound(a.shape[1], a, x)).all()), w


def _check(A, X, Q, bound=_bound):
    for w in _kinds(A, X.shape[1]):
        _check_one(w, A, X, Q, bound)


@pytest.mark.parametrize("rows,n,l,pad,off", SHAPES)
@pytest.mark.parametrize("mean", [0.0, 0.5])
def test_half_products(rows, n, l, pad, off, mean):
    dev = need_gpu()
    print(f"[case] half rows={rows} n={n} l={l} pad={pad} off={off} mean={mean}", flush=True)
    _check(*_inputs(rows, n, l, pad, off, dev, mean))


def _log_uniform(shape, lo, hi, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(77)
    return 10.0 ** (lo + (hi - lo) * torch.rand(shape, generator=g, device=dev))


def _graded(A, X, Q):            # columns over 24 decades, undone by the panel; rows likewise
    d, e = torch.logspace(-12, 12, A.shape[1], device=A.device), torch.logspace(-9, 9, A.shape[0], device=A.device)
    p = torch.randperm(len(d), generator=torch.Generator().manual_seed(5)).to(A.device)
    A *= d[p]
    X /= d[p][:, None]
    A *= e[:, None]
    Q /= e[:, None]


def _outliers(A, X, Q):          # large columns and rows of A where a column of the panel is zero, or small
    A[:, ::37] *= 1e7
    A[::41] *= 1e7
    X[::37, 0], X[::37, 3] = 0.0, X[::37, 3] * 1e-9
    Q[::41, 0], Q[::41, 3] = 0.0, Q[::41, 3] * 1e-9


def _few_outliers(A, X, Q):      # one element in a workgroup's part
    A[100, 200] = 1e9
    A[A.shape[0] - 1, A.shape[1] - 1] = -1e12
    X[200], Q[100] = 0.0, 0.0


def _any_range(A, X, Q):         # 30 decades without order
    A *= _log_uniform(A.shape, -30, 0, A.device)


def _panel_any_range(A, X, Q):
    X *= _log_uniform(X.shape, -20, 0, X.device)
    Q *= _log_uniform(Q.shape, -20, 0, Q.device)


def _indicators(A, X, Q):        # sums over groups of columns, one group of large numbers
    A[:, ::5] *= 1e8
    A[::5] *= 1e8
    for P in (X, Q):
        k = torch.arange(P.shape[0], device=P.device)
        P.zero_()
        P[k, k % 5 % P.shape[1]] = 1.0


def _blocks(A, X, Q):            # rows of A that only meet the small part of the panel, cut within a step
    h, k = A.shape[0] // 2 + 5, A.shape[1] // 2 + 5
    A[:h, k:], A[h:, :k] = 0.0, 0.0
    X[k:] *= 1e-9
    Q[h:] *= 1e-9


def _sparse(A, X, Q):            # a few numbers in a row, and none
    g = torch.Generator(device=A.device)
    g.manual_seed(9)
    A *= torch.rand(A.shape, generator=g, device=A.device) < 0.002
    A[7], A[:, 9] = 0.0, 0.0


def _zeros(A, X, Q):
    A[64:128, :], A[:, 64:200] = 0.0, 0.0
    X[64:200], Q[64:128] = 0.0, 0.0
    X[:, 1], Q[:, 1] = 0.0, 0.0


@pytest.mark.parametrize("change", [_graded, _outliers, _few_outliers, _any_range, _panel_any_range, _indicators, _blocks, _sparse, _zeros])
@pytest.mark.parametrize("rows,n,l,pad,off", [SHAPES[3], SHAPES[6], SHAPES[9], SHAPES[12]])
def test_half_products_of_every_range(rows, n, l, pad, off, change):
    """Each entry to the scale of the products it is made of, as with plain fp32 arithmetic."""
    dev = need_gpu()
    print(f"[case] half range {change.__name__} rows={rows} n={n} l={l}", flush=True)
    A, X, Q = _inputs(rows, n, l, pad, off, dev)
    change(A, X, Q)
    # small products may be subnormal (2^-149 apart, half of that for each of the partial sums)
    _check(A, X, Q, lambda K, a, x: _bound(K, a, x) + 2.0 ** -149 * K / 32)


# Sums of numbers that one scale per 64 loses, where the large ones beside them meet nothing.  a: some rows, x: one column of the panel.
def _covered(a, x, t):           # a large number and three small ones in every other four, the rest zero
    a.zero_()
    for i in range(4):
        a[:, i::8] = 1.0 if i == 0 else t
    x.copy_(x.sign())
    x[::8] = 0.0


def _selected(a, x, t):          # one number in 64, which meets a small one
    a.zero_()
    a[:, 5::64] = 1.0
    x[5::64] *= t


def _weak_fours(a, x, t):        # a number in every four that is large enough by itself, against a small entry
    a.copy_(a.sign() * t)
    a[:, 1::4] = 2.0 ** -16
    a[:, ::64] = 1.0
    x.copy_(x.sign())
    x[1::4] = 2.0 ** -9
    x[::64] = 0.0


def _at_the_limit(a, x, t):      # what the two tests of a step just let pass, for a panel with largest entries of 8
    k = torch.arange(a.shape[1], device=a.device) % 64
    a.copy_(a.sign() * t)
    a[:, (k % 2 == 0) & (k < 40)] = 2.0 ** -6
    a[:, k == 40] = 1.0
    x.copy_(x.sign() * 8.0)
    x[(k % 2 == 0) & (k < 20) | (k == 40)] = 0.0
    x[(k % 2 == 0) & (k >= 20) & (k < 40)] = 2.0 ** -6


@pytest.mark.parametrize("pattern", [_covered, _selected, _weak_fours, _at_the_limit])
@pytest.mark.parametrize("t", [2.0 ** -20, 2.0 ** -26, 2.0 ** -30, 2.0 ** -36, 2.0 ** -42])
@pytest.mark.parametrize("rows,n,l,pad,off", [SHAPES[3], SHAPES[8], SHAPES[12]])
def test_half_products_of_numbers_beside_larger_ones(rows, n, l, pad, off, pattern, t):
    dev = need_gpu()
    print(f"[case] half beside {pattern.__name__} {t} rows={rows} n={n} l={l}", flush=True)
    A, X, Q = _inputs(rows, n, l, pad, off, dev)
    X.clamp_(-8.0, 8.0)
    Q.clamp_(-8.0, 8.0)
    before = A.clone()
    for w in _kinds(A, l):
        A.copy_(before)
        a, x = (A, X) if w == 0 else (A.T, Q)
        rr = torch.tensor([1, 40, a.shape[0] // 2, a.shape[0] - 1], device=dev)
        picked, column = a[rr], x[:, 0].clone()
        pattern(picked, column, t)
        a[rr], x[:, 0] = picked, column
        _check_one(w, A, X, Q, lambda K, a_, x_: _bound(K, a_, x_) + 2.0 ** -149 * K / 32)


def _unsampled(count, row, steps):
    """The steps in which the packing's sample of A has not got this row."""
    return [c for c in range(steps) if (row - c * 2654435761) % count >= 64]


@pytest.mark.parametrize("rows,n,l,pad,off", [SHAPES[3], (16449, 257, 48, 0, 0), SHAPES[7], SHAPES[9], SHAPES[10], SHAPES[12]])
@pytest.mark.parametrize("places", ["one", "ends", "ten steps", "all steps", "all rows"])
def test_half_products_with_rare_outliers(rows, n, l, pad, off, places):
    """Rows that are left out of a step and added in fp32 leave all others bit for bit as they are.  (All steps of a row, or two of all
    rows of the last tile, are more than a wave keeps: then only the results of that tile may change.)"""
    dev = need_gpu()
    print(f"[case] half outliers {places} rows={rows} n={n} l={l}", flush=True)
    A, X, Q = _inputs(rows, n, l, pad, off, dev)
    for P in (X, Q):
        P[5::64] = P[5::64].sign()
        P[5::64, 0] = 0.0
    before = A.clone()
    for w in _kinds(A, l):
        A.copy_(before)
        plain = B.brsvd_gemm_an(A, X) if w == 0 else B.brsvd_gemm_at(A, Q)
        a = A if w == 0 else A.T
        count, K = a.shape
        steps = K // 64 + (K % 64 > 5)
        if places == "one":
            at = [(count // 2, _unsampled(count, count // 2, steps)[steps // 2])]
        elif places == "ends":
            at = [(r, c) for r in (0, count - 2, count - 1) for c in _unsampled(count, r, steps)[::max(1, steps - 2)]]
            at += [(r, steps - 1) for r in (count - 2, count - 1) if steps - 1 in _unsampled(count, r, steps)]
        elif places == "ten steps":
            at = [(count - 1, c) for c in _unsampled(count, count - 1, steps)[:10]]
        elif places == "all steps":
            at = [(count - 1, c) for c in _unsampled(count, count - 1, steps)]
        else:
            at = [(r, c) for r in range((count - 1) // 256 * 256, count) for c in _unsampled(count, r, steps)[2:4]]
        for r, c in at:
            a[r, 64 * c + 5] = 1e9
        _check_one(w, A, X, Q, _bound)
        got = B.brsvd_gemm_an(A, X) if w == 0 else B.brsvd_gemm_at(A, Q)
        same = torch.ones(count, dtype=torch.bool, device=dev)
        same[[r for r, _ in at]] = False
        if places.startswith("all"):
            same[(count - 1) // 256 * 256:] = False
        assert torch.equal(got[same], plain[same])


@pytest.mark.parametrize("scale_a,scale_x", [(1e-33, 1e28), (1e-41, 1e35), (1e30, 1e-37), (1e28, 1e-41), (1e-20, 1e-17), (1e30, 1e5)])
def test_half_products_at_any_exponent(scale_a, scale_x):
    dev = need_gpu()
    A, X, Q = _inputs(*SHAPES[3][:3], 0, 0, dev)
    A.mul_(scale_a)
    _check(A, X * scale_x, Q * scale_x, lambda K, a, x: _bound(K, a, x) + 2.0 ** -149 * K / 32)


@pytest.mark.parametrize("rows,n,l,pad,off", [SHAPES[3], (600, 16500, 161, 0, 0), (16500, 600, 273, 0, 0), SHAPES[12]])
def test_half_products_not_finite(rows, n, l, pad, off):
    _not_finite(rows, n, l, pad, off)


def test_half_products_repeat_bit_for_bit():
    """Also where some workgroups give up and redo their part."""
    dev = need_gpu()
    A, X, Q = _inputs(*SHAPES[3][:3], 0, 0, dev)
    _few_outliers(A, X, Q)
    first = B.brsvd_gemm_an(A, X), B.brsvd_gemm_at(A, Q)
    for _ in range(3):
        assert torch.equal(B.brsvd_gemm_an(A, X), first[0]) and torch.equal(B.brsvd_gemm_at(A, Q), first[1])


def test_half_products_with_more_workgroups_than_flags():
    """A workgroup beyond the 4096th does its part again by itself: the results of all others stay as they are, bit for bit."""
    dev = need_gpu()
    rows, n, l = 1060000, 1472, 48
    A, X = torch.randn(rows, n, generator=torch.Generator(device=dev).manual_seed(4), device=dev), _inputs(1, n, l, 0, 0, dev)[1]
    assert 0 in _kinds(A, l)
    plain = B.brsvd_gemm_an(A, X)
    steps = [c for c in range(n // 64) if all((rows - i - c * 2654435761) % rows >= 64 for i in range(1, 9))]
    for i in range(1, 9):                # more than a wave keeps
        A[rows - i, [64 * c for c in steps]] = 1e9
    got = B.brsvd_gemm_an(A, X)
    assert torch.equal(got[:4096 * 256], plain[:4096 * 256])
    tail = slice(rows - 300, rows)
    err = (got[tail].double() - A[tail].double() @ X.double()).abs()
    assert bool((err <= _bound(n, A[tail], X)).all())


@pytest.mark.parametrize("w,rows,n,l,most", [
    (0, 70000, 1409, 110, 1.05), (1, 1472, 60000, 110, 1.05), (0, 60000, 1800, 110, 1.0), (1, 1800, 60000, 110, 1.0), (0, 16000, 6000, 97, 1.0),
    (0, 1000, 16390, 110, 1.0), (1, 16390, 1000, 110, 1.0), (0, 8192, 12000, 60, 1.0), (1, 89083, 2783, 97, 0.9), (0, 20000, 20000, 110, 0.9)])
def test_half_products_are_as_accurate_as_six_bf16_ones(w, rows, n, l, most):
    """From the lines on where they are taken (at the shortest one both are alike: 2^-24 of each product is lost in place of half of 44 rounded
    additions).  The last column decides: one number in 64 leaves all of them to bf16."""
    dev = need_gpu()
    g = torch.Generator(device=dev).manual_seed(12)
    A = torch.randn(rows, n, generator=g, device=dev)
    P = torch.randn(n if w == 0 else rows, l, generator=g, device=dev)
    assert B.brsvd_gemm_is_split(w, rows, n, l) and B.brsvd_gemm_split_parts(w, rows, n, l) == 2
    product = B.brsvd_gemm_an if w == 0 else B.brsvd_gemm_at
    exact = (A.double() @ P.double() if w == 0 else A.double().T.contiguous() @ P.double())[:, :l - 1]
    error = []
    for sparse in (False, True):
        if sparse:
            P[:, l - 1] = 0.0
            P[::64, l - 1] = 1.0
        error.append(float((product(A, P)[:, :l - 1].double() - exact).norm() / exact.norm()))
    print(f"[case] half {w} {rows}x{n} l={l} errors {error[0]:.3e} {error[1]:.3e}", flush=True)
    assert error[0] != error[1] and error[0] <= most * error[1]
