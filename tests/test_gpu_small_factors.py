"""The l x l factors at the edges of their tiles and of the kernels' ranges: Cholesky factor and inverse behind the
orthonormalisation (16 x 16 tiles, in LDS up to 128, in global memory above), and the Jacobi SVD (row blocks of 16; row
rotations up to 16 and for 33 to 48 rows, one workgroup up to 32 rows, a workgroup per block pair otherwise)."""
import threading
import time

import numpy as np
import pytest
import torch

import paper_1706_07191_amd as B
from paper_1706_07191_amd import synth
from tests.gpu_util import EPS32, need_gpu

pytestmark = pytest.mark.gpu

EDGES = [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 127, 128, 129, 144, 161, 272, 512]


def _panel(rows, l, decay, seed):
    g = torch.Generator().manual_seed(seed)
    s = torch.exp(-torch.arange(l, dtype=torch.float64) * (np.log(decay) / max(l, 2)))
    mix = torch.linalg.qr(torch.randn(l, l, generator=g, dtype=torch.float64))[0]
    return ((torch.randn(rows, l, generator=g, dtype=torch.float64) * s) @ mix).float()


@pytest.mark.parametrize("l", EDGES)
@pytest.mark.parametrize("method", [B.BRSVD_ORTH_AUTO, B.BRSVD_ORTH_TSQR])
def test_orthonormalisation_and_its_factor(l, method):
    dev = need_gpu()
    print(f"[case] orth l={l} method={method}", flush=True)
    rows = 3 * l + 70
    P = _panel(rows, l, 30.0, l)
    Q, R, _ = B.brsvd_orth(P.to(dev), method=method, want_R=True)
    Q, R = Q.double().cpu(), R.cpu()
    eye = torch.eye(l, dtype=torch.float64)
    # Q is stored in fp32: each entry of Q^T Q carries the rounding of rows products of entries around rows^-1/2 (random
    # signs), and the product P R^-1 that of l terms; P = Q R holds to the same, times the size of R's columns
    assert float((Q.T @ Q - eye).abs().max()) <= 8 * EPS32 * np.sqrt(l)
    assert float((Q @ R - P.double()).abs().max()) <= 16 * EPS32 * np.sqrt(l) * float(P.double().norm(dim=0).max() / np.sqrt(rows) * 4)
    assert bool((torch.tril(R, -1) == 0).all())
    if method == B.BRSVD_ORTH_AUTO:
        assert bool((torch.diagonal(R) > 0).all())


def test_zero_columns_are_clamped():
    """Columns of zeros: their pivots are clamped in the first sweep and refused in the last one, the fallback takes over or
    the call says so; nothing is left undefined."""
    dev = need_gpu()
    P = _panel(500, 40, 10.0, 5)
    P[:, 17] = 0
    try:
        Q, R, fb = B.brsvd_orth(P.to(dev), want_R=True)
        assert bool(torch.isfinite(Q).all()) and bool(torch.isfinite(R).all())
    except B.BrsvdError as e:
        assert e.status == B.BRSVD_ERR_ORTH_BREAKDOWN


@pytest.mark.parametrize("l", EDGES)
@pytest.mark.parametrize("cond", [1e2, 1e8])
def test_small_svd(l, cond):
    dev = need_gpu()
    print(f"[case] small_svd l={l} cond={cond}", flush=True)
    g = torch.Generator().manual_seed(1000 + l)
    s = torch.logspace(0, -np.log10(cond), l, dtype=torch.float64)
    q = [torch.linalg.qr(torch.randn(l, l, generator=g, dtype=torch.float64))[0] for _ in range(2)]
    R = torch.linalg.qr((q[0] * s) @ q[1])[1]
    S, U, V, sweeps = (x.cpu() if isinstance(x, torch.Tensor) else x for x in B.brsvd_small_svd(R.to(dev).contiguous()))
    ref = torch.linalg.svdvals(R)
    eye = torch.eye(l, dtype=torch.float64)
    eps = 2.0 ** -52
    assert sweeps <= 20 and bool((S[:-1] >= S[1:]).all())
    # LAPACK's values are good to a few eps of the largest one; rotations act on rows of l entries
    assert float((S - ref).abs().max()) <= 40 * eps * np.sqrt(l)
    # cosines far below 1e-13 are left; U = R V / s carries them times s_1 / s_i
    assert float((V.T @ V - eye).abs().max()) <= 4e-13
    assert float((U.T @ U - eye).abs().max()) <= 4e-13 * cond * 10
    assert float(((U * S) @ V.T - R).abs().max()) <= 1e-12


@pytest.mark.parametrize("l", [2, 3, 16, 17, 20, 21])
def test_small_svd_at_the_ends_of_the_row_rotations(l):
    """Row rotations up to 16 rows, one block pair from 17 on."""
    for cond in (1e2, 1e8):
        test_small_svd(l, cond)


@pytest.mark.parametrize("l", [13, 16, 17, 24, 33, 40, 41, 44, 48, 49, 66, 72, 79])
def test_small_svd_where_rows_and_blocks_meet(l):
    """Row rotations up to 16 and from 33 to 48 rows, block pairs otherwise; well-conditioned, nearly rank deficient, and with all
    entries so small that the squares of squared norms are below the smallest double."""
    for cond in (1e2, 1e8):
        test_small_svd(l, cond)
    dev = need_gpu()
    g = torch.Generator().manual_seed(l)
    R = torch.linalg.qr(torch.randn(3 * l, l, generator=g, dtype=torch.float64))[1].contiguous()
    ref = torch.linalg.svdvals(R)
    S, U, V, _ = (x.cpu() if isinstance(x, torch.Tensor) else x for x in B.brsvd_small_svd((R * 2.0 ** -440).to(dev)))
    assert float((S * 2.0 ** 440 - ref).abs().max()) <= 40 * 2.0 ** -52 * np.sqrt(l) * float(ref[0])
    assert float((V.T @ V - torch.eye(l, dtype=torch.float64)).abs().max()) <= 4e-13


def _singular_values_long(R):
    """One-sided Jacobi on the rows in 80-bit arithmetic."""
    W, l = R.numpy().astype(np.longdouble), R.shape[0]
    n = l + l % 2
    W = np.vstack((W, np.zeros((n - l, l), np.longdouble)))
    for _ in range(30):
        worst = 0.0
        for step in range(n - 1):
            i = np.arange(1, n // 2)
            a, b = np.r_[n - 1, (step + i) % (n - 1)], np.r_[step, (step - i) % (n - 1)]
            x, y = W[a], W[b]
            al, be, ga = (x * x).sum(1), (y * y).sum(1), (x * y).sum(1)
            on = ga * ga > np.longdouble(1e-36) * al * be
            ga, tau = np.where(on, ga, 1), np.where(on, be - al, 0)
            worst = max(worst, float(np.max(np.where(on, ga * ga / np.where(on, al * be, 1), 0))))
            t = np.where(on, 2 * ga / (np.abs(tau) + np.hypot(tau, 2 * ga)) * np.where(tau < 0, -1, 1), 0)
            c = 1 / np.sqrt(1 + t * t)
            W[a], W[b] = c[:, None] * x - (c * t)[:, None] * y, (c * t)[:, None] * x + c[:, None] * y
        if worst < 1e-18:
            break
    return np.sort(np.sqrt((W * W).sum(1)))[::-1][:l]


@pytest.mark.parametrize("l", [20, 40, 60, 110, 272])
@pytest.mark.parametrize("decades", [12, 30, 60])
def test_small_svd_of_graded_rows(l, decades):
    """Rows that shrink by many decades, times a well-conditioned matrix: rotations leave every singular value, also the smallest,
    its own relative accuracy."""
    dev = need_gpu()
    print(f"[case] graded l={l} decades={decades}", flush=True)
    g = torch.Generator().manual_seed(l + decades)
    Bm = torch.eye(l, dtype=torch.float64) + 0.3 * torch.randn(l, l, generator=g, dtype=torch.float64) / np.sqrt(l)
    R = torch.logspace(0, -decades, l, dtype=torch.float64)[:, None] * Bm
    S, U, V, sweeps = (x.cpu() if isinstance(x, torch.Tensor) else x for x in B.brsvd_small_svd(R.to(dev).contiguous()))
    ref = _singular_values_long(R)
    rel = float(np.max(np.abs(S.numpy().astype(np.longdouble) - ref) / ref))
    print(f"[case] sweeps={sweeps} rel={rel:.2e}", flush=True)
    # about l rotations a sweep touch a row, each with a rounding of eps of the row it changes; as a random walk, times the
    # condition of the matrix with its rows scaled to one (4 here)
    assert rel <= 4 * 2.0 ** -52 * np.sqrt(l * sweeps) * 4
    assert float((V.T @ V - torch.eye(l, dtype=torch.float64)).abs().max()) <= 4e-13


@pytest.mark.parametrize("l", [16, 30, 40, 48, 97, 200, 400])
@pytest.mark.parametrize("q", [0, 1])
@pytest.mark.parametrize("ratio", [1e-4, 1e-6])
@pytest.mark.parametrize("f64", [False, True])
def test_vectors_of_steep_spectra(l, q, ratio, f64):
    """SVDs whose small factor has a condition of 1e4 and 1e6: V = W_B (R V_R / s) carries a cosine that the iteration leaves
    between rows i and j times s_i / s_j, so block pairs may only be passed over by a bar that knows the norms."""
    dev = need_gpu()
    print(f"[case] steep spectrum l={l} q={q} ratio={ratio} f64={f64}", flush=True)
    dt = torch.float64 if f64 else torch.float32
    m, n = 3 * l + 300, 3 * l + 200
    s = torch.exp(-torch.arange(2 * l, dtype=torch.float64) * (np.log(1 / ratio) / l))
    A = synth.exact_spectrum_matrix(m, n, s, l + q, dt).contiguous()
    h = B.brsvd_create(B.make_params(m, n, l - 10, 10, q, dtype=B.BRSVD_DTYPE_F64 if f64 else B.BRSVD_DTYPE_F32))
    try:
        U, S, Vt, st = B.brsvd_run(h, A.to(dev), synth.gaussian(n, l, 5, dtype=dt).to(dev))
    finally:
        B.brsvd_destroy(h)
    eye = torch.eye(l, dtype=torch.float64, device=dev)
    # fp32: entries rounded to 2^-24 of themselves leave a random matrix of variance 2^-48 in X^T X, of norm 2 sqrt(l) 2^-24.
    # fp64: a row meets l rotations in each of up to ten sweeps, as a random walk sqrt(10 l) roundings; twice over for what R V / s adds
    tol = 4 * 2 * np.sqrt(l) * np.sqrt(10 * l) * 2.0 ** -53 if f64 else 2 * np.sqrt(l) * 2.0 ** -24
    if f64 and (l <= 16 or 33 <= l <= 48):          # row rotations leave cosines below 1e-16, of each row with l others
        tol += l * 1e-16 / ratio
    for X in (U.double(), Vt.double().T):
        assert float(torch.linalg.norm(X.T @ X - eye, 2)) <= tol
    assert 0.3 * ratio < float(S[-1] / S[0]) < 3 * ratio and st["orth_fallbacks"] == 0


@pytest.mark.parametrize("l", [17, 24, 32])
@pytest.mark.parametrize("d", [1e-8, 1e-9])
def test_small_svd_of_two_parallel_rows(l, d):
    """Two rows e_i and e_i + d e_j in a random basis, the others orthogonal: the first rotation leaves nothing on the Gram matrix it was
    taken from, but the rows it gives have a cosine of d / 2, which U = R V / s shows times s_1 / s_l.  The end of the iteration has
    to be seen on a Gram matrix of the rows themselves."""
    dev = need_gpu()
    print(f"[case] parallel rows l={l} d={d}", flush=True)
    eye = torch.eye(l, dtype=torch.float64)
    for i, j in ((0, 8), (0, 16), (2, 3)):
        for seed in range(60):
            R = torch.diag(torch.linspace(3, 5, l, dtype=torch.float64))
            R[j, j], R[i, i], R[j, i] = d, 1, 1
            R = R @ torch.linalg.qr(torch.randn(l, l, generator=torch.Generator().manual_seed(seed), dtype=torch.float64))[0]
            S, U, V, _ = (x.cpu() if isinstance(x, torch.Tensor) else x for x in B.brsvd_small_svd(R.to(dev).contiguous()))
            assert float((V.T @ V - eye).abs().max()) <= 4e-13, (i, j, seed)
            # U = R V / s: the rounding of R V, of rows of norm s_1, over s_l
            assert float((U.T @ U - eye).abs().max()) <= 8 * 2.0 ** -53 * float(S[0] / S[-1]), (i, j, seed)


def test_small_svd_of_equal_and_zero_values():
    dev = need_gpu()
    for l in (16, 30, 40, 100, 160):
        g = torch.Generator().manual_seed(l)
        Q = torch.linalg.qr(torch.randn(l, l, generator=g, dtype=torch.float64))[0]
        S, U, V, _ = B.brsvd_small_svd(Q.to(dev).contiguous())             # all singular values equal
        assert float((S.cpu() - 1).abs().max()) <= 1e-13
        R = torch.linalg.qr(torch.randn(l, l, generator=g, dtype=torch.float64))[1]
        R[l // 2:] = 0                                                     # rank l / 2
        S = B.brsvd_small_svd(R.to(dev).contiguous())[0].cpu()
        ref = torch.linalg.svdvals(R)
        assert float((S - ref).abs().max()) <= 1e-13 * float(ref[0])
        assert bool((B.brsvd_small_svd(torch.zeros(l, l, dtype=torch.float64, device=dev))[0] == 0).all())


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), float("-inf"), 1e160])
@pytest.mark.parametrize("l", [30, 40, 60, 110, 160])
def test_small_svd_with_a_row_that_is_not_finite(l, bad):
    """The row keeps its own norm (infinite, or NaN before all others) and the other rows are orthogonalised as if it were not
    there; nothing an earlier call left in the scratch comes out."""
    dev = need_gpu()
    g = torch.Generator().manual_seed(l)
    R = torch.linalg.qr(torch.randn(2 * l, l, generator=g, dtype=torch.float64))[1].contiguous()
    for static in (False, True):
        before = B.brsvd_small_svd(R.to(dev), static=static)[0].cpu()
        Rb = R.clone()
        Rb[3, 7] = bad
        S, U, V, _ = (x.cpu() if isinstance(x, torch.Tensor) else x for x in B.brsvd_small_svd(Rb.to(dev), static=static))
        assert bool(S[0].isnan()) if bad != bad else float(S[0]) == float("inf")
        ref = torch.linalg.svdvals(torch.cat((R[:3], R[4:])))
        assert float((S[1:] - ref).abs().max()) <= 1e-12 * float(ref[0])
        eye = torch.eye(l - 1, dtype=torch.float64)
        assert float((V[:, 1:].T @ V[:, 1:] - eye).abs().max()) <= 4e-13
        again = B.brsvd_small_svd(R.to(dev), static=static)[0].cpu()
        assert torch.equal(before, again)


def test_block_pairs_on_several_streams():
    """Calls whose workgroups wait for each other, at the same time on four streams (one host thread each: a call returns when
    its work is done) beside a stream of large products: every call ends and gives what it gives alone."""
    dev = need_gpu()
    g = torch.Generator().manual_seed(9)
    Rs = [torch.linalg.qr(torch.randn(l, l, generator=g, dtype=torch.float64))[1].to(dev).contiguous() for l in (81, 130, 200, 512)]
    alone = [B.brsvd_small_svd(R)[0].clone() for R in Rs]
    big = torch.randn(8192, 8192, device=dev)
    product = torch.empty_like(big)
    streams = [torch.cuda.Stream() for _ in Rs]
    busy = torch.cuda.Stream()
    outs = [tuple(torch.empty(s, dtype=torch.float64, device=dev) for s in (R.shape[0], R.shape, R.shape)) for R in Rs]
    nbytes = [B.lib().brsvd_small_svd_scratch_bytes(R.shape[0]) for R in Rs]
    scratch = [torch.empty(n, dtype=torch.uint8, device=dev) for n in nbytes]
    start = threading.Barrier(len(Rs) + 1)
    wrong, spans = [], [[] for _ in Rs]

    def calls(i):
        l = Rs[i].shape[0]
        for _ in range(5):
            start.wait(60)
            for _ in range(4 * 512 // l):
                t0 = time.perf_counter()
                st = B.lib().brsvd_small_svd(Rs[i].data_ptr(), l, *(o.data_ptr() for o in outs[i]), None, scratch[i].data_ptr(),
                                             nbytes[i], streams[i].cuda_stream)
                spans[i].append((t0, time.perf_counter()))
                if st != B.BRSVD_OK:
                    wrong.append((l, st))
            with torch.cuda.stream(streams[i]):
                if not bool(torch.equal(alone[i], outs[i][0])):
                    wrong.append((l, "values"))

    threads = [threading.Thread(target=calls, args=(i,)) for i in range(len(Rs))]
    torch.cuda.synchronize()
    for th in threads:
        th.start()
    for _ in range(5):
        with torch.cuda.stream(busy):          # some 40 ms of work, in the queue before the calls
            for _ in range(5):
                torch.mm(big, big, out=product)
        start.wait(60)
    for th in threads:
        th.join(60)
    torch.cuda.synchronize()
    assert not wrong and not any(th.is_alive() for th in threads)
    # the calls did run beside each other
    met = sum(a0 < b1 and b0 < a1 for a0, a1 in spans[3] for b0, b1 in spans[0])
    print(f"[case] {met} calls of l=81 beside a call of l=512", flush=True)
    assert met > 0


@pytest.mark.parametrize("l", [49, 81, 112, 134, 161, 257, 512])
def test_workgroups_see_each_others_rows(l):
    """The rows travel between workgroups through global memory: a fixed order of operations, so every call gives the same
    bits and a row read too early shows at once.  Full rank and rank l - 10 (rows of rounding noise)."""
    dev = need_gpu()
    g = torch.Generator().manual_seed(l)
    A = torch.randn(2 * l, l, generator=g, dtype=torch.float64)
    B10 = torch.randn(2 * l, l - 10, generator=g, dtype=torch.float64) @ torch.randn(l - 10, l, generator=g, dtype=torch.float64)
    for M in (A, B10):
        R = torch.linalg.qr(M)[1].to(dev).contiguous()
        first = [x.clone() for x in B.brsvd_small_svd(R)[:3]]
        assert float(((first[1] * first[0]) @ first[2].T - R).abs().max()) <= 1e-12 * float(first[0][0])
        for _ in range(60):
            again = B.brsvd_small_svd(R)
            assert all(bool(torch.equal(a.nan_to_num(), b.nan_to_num())) for a, b in zip(first, again))


@pytest.mark.parametrize("l", [1, 16, 17, 33, 48])
@pytest.mark.parametrize("rows", [51, 1000, 131089])
def test_narrow_panels_times_their_factors(l, rows):
    """Tiles of 16 rows that end in a remainder, and more of them than waves (131072 rows): the factors applied by the
    orthonormalisation (whole padded panels) and by the lift (l columns)."""
    dev = need_gpu()
    print(f"[case] apply l={l} rows={rows}", flush=True)
    P = _panel(rows, l, 30.0, 11).to(dev)
    Q, R, _ = B.brsvd_orth(P.clone(), want_R=True)
    Pd, Qd = P.double(), Q.double()
    # two sweeps, each a product over l terms with a rounding per term
    assert float((Qd @ R.double() - Pd).abs().max() / Pd.abs().max()) <= 4 * (l + 2) * EPS32
    assert float((Qd.T @ Qd - torch.eye(l, device=dev, dtype=torch.float64)).abs().max()) <= 4 * (l + 2) * EPS32
    A = (P @ _panel(l + 40, l, 3.0, 12).to(dev).T).contiguous()
    h = B.brsvd_create(B.make_params(rows, l + 40, l, 0, 1))
    try:
        U, S, Vt, _ = B.brsvd_run(h, A, torch.randn(l + 40, l, generator=torch.Generator().manual_seed(3)).to(dev))
    finally:
        B.brsvd_destroy(h)
    err = (U.double() * S.double()) @ Vt.double() - A.double()
    assert float(err.norm() / A.double().norm()) <= 1e-5            # rank l exactly, fp32 products
    assert float((U.double().T @ U.double() - torch.eye(l, device=dev, dtype=torch.float64)).abs().max()) <= 1e-5
