"""The block-local scheme of Alg. 2 (brsvd_run_alg2) and the device-side Gaussian generator against
their oracles."""
import numpy as np
import pytest
import torch

import paper_1706_07191_amd as B
from oracle import brsvd_oracle as O
from oracle import philox as PX
from paper_1706_07191_amd import synth
from tests.gpu_util import EPS32, ORTH_TOL, RECON_RTOL, SIGMA_RTOL, need_gpu, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed,rows,cols,row0", [(1, 1000, 30, 0), (2 ** 40 + 17, 257, 110, 12345), (99, 5, 3, 7),
                                                   (7, 1, 1, 0), (2 ** 63 + 5, 64, 272, 2 ** 31)])
def test_philox_normal_matches_oracle(seed, rows, cols, row0):
    """Same counters, same key, same transform: the integer part is exact, the fp32 Box-Muller agrees
    with the fp64 one to a few ulp of fp32."""
    need_gpu()
    g = B.brsvd_philox_normal(seed, rows, cols, row0).double().cpu().numpy()
    o = PX.philox_normal(seed, rows, cols, row0)
    assert np.max(np.abs(g - o) / (1.0 + np.abs(o))) <= 1e-6
    # a window equals the slice of a larger draw, bit for bit
    if rows >= 5:
        w = B.brsvd_philox_normal(seed, 3, cols, row0 + 2).cpu().numpy()
        np.testing.assert_array_equal(w, B.brsvd_philox_normal(seed, rows, cols, row0).cpu().numpy()[2:5])


def _figures(A, Om, cfg, b, U, S, Vt):
    Uo, so, Vto = O.brsvd_alg2(A, Om, cfg.k, cfg.p, cfg.q, row_block=b)
    Ug, sg, Vg = U.double().cpu().numpy(), S.double().cpu().numpy(), Vt.double().cpu().numpy()
    k = cfg.k
    f = {"sigma_rel": float(np.max(np.abs(sg[:k] - so[:k]) / so[:k])), "orthU": O.orth_defect(Ug),
         "orthV": O.orth_defect(Vg.T), "err_gpu": O.recon_error(A, Ug, sg, Vg, k=k),
         "err_oracle": O.recon_error(A, Uo, so, Vto, k=k),
         "growth": float((so[0] / so[k - 1]) ** (2 * cfg.q + 1))}
    assert np.all(np.diff(sg) <= 0) and np.all(sg >= 0)
    return f, sg, so


@pytest.mark.parametrize("name,m,n,b,q", [("C1", 2000, 1000, 512, 2), ("C1", 1500, 800, 333, 0), ("C1", 1500, 800, 333, 1),
                                           ("C3", 4000, 3000, 1024, 1), ("C4", 3000, 3500, 900, 1),
                                           ("C4", 3000, 3500, 3000, 1)])
def test_alg2_matches_oracle(name, m, n, b, q):
    """Same A and Omega on both sides; spectra whose (s_1/s_k)^(2q+1) stays below about 1e6, so that the
    unorthonormalised block-local power iteration is still resolved in fp32."""
    dev = need_gpu()
    cfg = synth.CONFIGS[name].scaled(m, n, b)
    cfg.q = q
    A = cfg.make_A()
    Om = synth.gaussian(m, cfg.l, cfg.seed + 77)
    h = B.brsvd_create(B.make_params(m, n, cfg.k, cfg.p, q, row_block=b))
    try:
        U, S, Vt, st = B.brsvd_run_alg2(h, A.to(dev), cfg.l, Omega=Om.to(dev))
    finally:
        B.brsvd_destroy(h)
    f, _, _ = _figures(A.numpy(), Om.numpy(), cfg, b, U, S, Vt)
    note(f"[alg2 {name} {m}x{n} b={b} q={q}] " + " ".join(f"{k_}={v:.3e}" for k_, v in f.items()))
    # A lives in device memory: the kernels read every block 2q+1 times in the first sweep and once in the second;
    # only a host-resident A is read (over the host link) twice whatever q is
    assert st["passes_over_A"] == 2 * q + 2 and st["orth_fallbacks"] == 0
    assert st["gemm_at_launches"] == st["n_blocks"] * (q + 1) and st["gemm_an_launches"] == st["n_blocks"] * q + 1
    assert f["sigma_rel"] <= SIGMA_RTOL
    assert f["orthU"] <= ORTH_TOL and f["orthV"] <= ORTH_TOL
    assert abs(f["err_gpu"] - f["err_oracle"]) <= RECON_RTOL * f["err_oracle"]


def test_alg2_on_device_omega_and_streaming():
    """Omega drawn by the library from a seed equals the oracle's draw of the same matrix; a host-resident A
    streamed block by block gives the in-core result up to fp32 summation order (the second sweep is one
    launch in core and one per block when streamed, with different split plans)."""
    dev = need_gpu()
    m, n, b = 2600, 1500, 640
    cfg = synth.CONFIGS["C4"].scaled(m, n, b)
    A = cfg.make_A()
    seed = 2 ** 33 + 12345
    Om = PX.philox_normal(seed, m, cfg.l)
    h = B.brsvd_create(B.make_params(m, n, cfg.k, cfg.p, cfg.q, row_block=b))
    try:
        U, S, Vt, st = B.brsvd_run_alg2(h, A.to(dev), cfg.l, seed=seed)
        U2, S2, Vt2, _ = B.brsvd_run_alg2(h, A.to(dev), cfg.l, seed=seed)
    finally:
        B.brsvd_destroy(h)
    assert torch.equal(S, S2) and torch.equal(U, U2) and torch.equal(Vt, Vt2)
    f, _, _ = _figures(A.numpy(), Om, cfg, b, U, S, Vt)
    note("[alg2 seeded] " + " ".join(f"{k_}={v:.3e}" for k_, v in f.items()))
    assert f["sigma_rel"] <= SIGMA_RTOL and f["orthU"] <= ORTH_TOL and f["orthV"] <= ORTH_TOL
    assert abs(f["err_gpu"] - f["err_oracle"]) <= RECON_RTOL * f["err_oracle"]
    Ah = A.pin_memory()
    h = B.brsvd_create(B.make_params(m, n, cfg.k, cfg.p, cfg.q, row_block=b, a_location=B.BRSVD_A_HOST_PINNED))
    try:
        Uh, Sh, Vth, sth = B.brsvd_run_alg2(h, Ah, cfg.l, seed=seed)
    finally:
        B.brsvd_destroy(h)
    assert sth["passes_over_A"] == 2 and sth["copy_seconds"] > 0
    assert sth["bytes_A_streamed"] == 2 * 4 * m * n and sth["bytes_A_read_by_kernels"] == (2 * cfg.q + 2) * 4 * m * n
    k = cfg.k
    assert float(torch.max(torch.abs(S - Sh)[:k] / S[:k])) <= 1e-5
    R1 = (U[:, :k].double() * S[:k].double()) @ Vt[:k].double()
    R2 = (Uh[:, :k].double() * Sh[:k].double()) @ Vth[:k].double()
    assert float(torch.linalg.norm(R1 - R2) / torch.linalg.norm(R1)) <= 1e-4


def test_alg2_fp32_limit_of_the_unorthonormalised_power_iteration():
    """Configuration-2 spectrum (s_i = 1/i, k = 100).  q = 1: (s_1/s_k)^3 = 1e6 is the edge of what fp32
    resolves, the top-k values agree to 1e-3.  q = 2: (s_1/s_k)^5 = 1e10 is far beyond it -- the sketch
    panel is numerically rank deficient (the Householder-tree fallback is taken) and only the leading
    directions survive; the result is still an orthonormal factorisation whose values never exceed the
    oracle's by more than rounding, and whose leading values match."""
    dev = need_gpu()
    m, n, b = 3000, 2500, 700
    out = {}
    for q in (1, 2):
        cfg = synth.CONFIGS["C2"].scaled(m, n, b)
        cfg.q = q
        A = cfg.make_A()
        Om = synth.gaussian(m, cfg.l, cfg.seed + 77)
        h = B.brsvd_create(B.make_params(m, n, cfg.k, cfg.p, q, row_block=b))
        try:
            U, S, Vt, st = B.brsvd_run_alg2(h, A.to(dev), cfg.l, Omega=Om.to(dev))
        finally:
            B.brsvd_destroy(h)
        f, sg, so = _figures(A.numpy(), Om.numpy(), cfg, b, U, S, Vt)
        note(f"[alg2 C2 q={q}] " + " ".join(f"{k_}={v:.3e}" for k_, v in f.items()) + f" fallbacks={st['orth_fallbacks']}")
        assert f["orthU"] <= ORTH_TOL and f["orthV"] <= ORTH_TOL
        out[q] = (f, sg, so)
    f, sg, so = out[1]
    assert f["sigma_rel"] <= 1e-3 and abs(f["err_gpu"] - f["err_oracle"]) <= RECON_RTOL * f["err_oracle"]
    f, sg, so = out[2]
    lead = (so / so[0]) ** 5 > 1e-4          # directions well above the fp32 floor of the sketch
    assert lead.sum() >= 5 and np.max(np.abs(sg[lead] - so[lead]) / so[lead]) <= 1e-3
    sv = np.linalg.svd(A.double().numpy(), compute_uv=False)
    assert np.all(sg <= sv[:sg.size] * (1 + 1e-5))
    assert f["err_oracle"] <= f["err_gpu"] <= 1.5 * f["err_oracle"]


def test_alg2_argument_errors():
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"].scaled(300, 200, 100)
    A = cfg.make_A().to(dev)
    h = B.brsvd_create(B.make_params(300, 200, cfg.k, cfg.p, cfg.q, row_block=100))
    try:
        with pytest.raises(B.BrsvdError):
            B.brsvd_run_alg2(h, A, cfg.l, lda=100)          # lda < n
        L = B.lib()
        assert L.brsvd_run_alg2(h, None, 200, 0, None, None, None, None, None) == B.BRSVD_ERR_ARG
        assert L.brsvd_philox_normal(1, 0, 0, 4, A.data_ptr(), None) == B.BRSVD_ERR_ARG
        assert L.brsvd_philox_normal(1, -1, 4, 4, A.data_ptr(), None) == B.BRSVD_ERR_ARG
    finally:
        B.brsvd_destroy(h)


def test_alg2_seeded_random_shapes():
    """Fifteen seeded random problems for the block-local scheme (q <= 1, gently decaying spectrum, so that the
    unorthonormalised block sketches stay resolved in fp32), Omega drawn on the device."""
    import random
    dev = need_gpu()
    rng = random.Random(2170607)
    for case in range(15):
        m = rng.choice([rng.randint(60, 400), rng.randint(400, 2500)])
        n = rng.choice([rng.randint(60, 400), rng.randint(400, 2500)])
        l = rng.randint(2, min(m, n, 48) - 1)
        p = rng.randint(0, min(l - 1, 8))
        k, q = l - p, rng.randint(0, 1)
        b = rng.randint(max(1, m // 6), m)
        sig = torch.tensor([0.97 ** i for i in range(min(m, n))], dtype=torch.float64)
        A = synth.lowrank_plus_noise(m, n, sig, 1e-3, 9400 + case)
        seed = 2 ** 35 + 1000 * case + 7
        Om = PX.philox_normal(seed, m, l)
        cfg = synth.Config(f"rand-alg2-{case}", m, n, k, p, q, b, min(m, n), lambda i: i, 1e-3, 9400 + case)
        print(f"[case {case}] m={m} n={n} k={k} p={p} q={q} b={b}", flush=True)
        h = B.brsvd_create(B.make_params(m, n, k, p, q, row_block=b))
        try:
            U, S, Vt, st = B.brsvd_run_alg2(h, A.to(dev), l, seed=seed)
        finally:
            B.brsvd_destroy(h)
        f, _, _ = _figures(A.numpy(), Om, cfg, b, U, S, Vt)
        note(f"[alg2 rand{case}] " + " ".join(f"{k_}={v:.3e}" for k_, v in f.items()))
        assert st["passes_over_A"] == (2 * q + 2) * (1 + st["orth_fallbacks"])
        assert f["sigma_rel"] <= SIGMA_RTOL and f["orthU"] <= ORTH_TOL and f["orthV"] <= ORTH_TOL
        assert abs(f["err_gpu"] - f["err_oracle"]) <= RECON_RTOL * f["err_oracle"]


def test_alg2_products_keep_all_bits():
    """The sketch of the block-local scheme is taken with operands of 24 bits, over long contractions too.  With q = 0 and one block it
    is A^T Omega; a panel with one more column, sparse enough that its product takes that route in any case, gives the same columns bit
    for bit.  Their condition is about 1e4, so that V would leave their span by 1e-3 if the sketch were rounded otherwise."""
    dev = need_gpu()
    m, n, l = 20000, 1500, 60
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    rnd = lambda *shape: torch.randn(*shape, generator=g, device=dev)
    A = (rnd(m, l) * torch.logspace(0, -4, l, device=dev)) @ rnd(l, n) + 1e-6 * rnd(m, n)
    Om = rnd(m, l)
    assert B.brsvd_gemm_is_split(1, m, n, l) and B.brsvd_gemm_split_parts(1, m, n, l) == 2
    h = B.brsvd_create(B.make_params(m, n, l - 10, 10, 0, row_block=m))
    try:
        _, _, Vt, _ = B.brsvd_run_alg2(h, A, l, Omega=Om)
    finally:
        B.brsvd_destroy(h)
    wide = torch.zeros(m, l + 1, device=dev)
    wide[:, :l] = Om
    wide[::64, l] = 1.0
    Q = B.brsvd_orth(B.brsvd_gemm_at(A, wide)[:, :l].contiguous())[0].double()
    V = Vt.double().T
    assert float((V - Q @ (Q.T @ V)).norm()) <= 2.0 * l * EPS32 * l ** 0.5


@pytest.mark.parametrize("seed", [1, 2])
def test_alg2_vectors_against_64_bits(seed):
    """Powers without re-orthonormalisation carry 64^3 = 2.6e5 from the first direction to the last, so the last vectors follow every change in
    the order of the fp32 sums; the whole stays at the same distance from the scheme in 64 bits, and every call gives the same bits."""
    dev = need_gpu()
    m, n, k, p, b = 9000, 3000, 90, 10, 4096
    l = k + p
    s = torch.exp(-torch.arange(1, 2 * l + 1, dtype=torch.float64) * (np.log(64.0) / l)).float()
    A = synth.lowrank_plus_noise(m, n, s, 1e-4, 10 * seed)
    Om = synth.gaussian(m, l, 10 * seed + 7)
    h = B.brsvd_create(B.make_params(m, n, k, p, 1, row_block=b))
    try:
        out = [B.brsvd_run_alg2(h, A.to(dev), l, Omega=Om.to(dev))[:3] for _ in range(2)]
    finally:
        B.brsvd_destroy(h)
    assert all(torch.equal(x, y) for x, y in zip(*out))
    A, Om = A.to(dev).double(), Om.to(dev).double()
    Y = sum(A[r:r + b].T @ (A[r:r + b] @ (A[r:r + b].T @ Om[r:r + b])) for r in range(0, m, b))
    Q = torch.linalg.qr(Y)[0]
    W, R = torch.linalg.qr(A @ Q)
    u, sv, vt = torch.linalg.svd(R.cpu())
    U, S, Vt = (x.double() for x in out[0])
    Ue, Vte = W @ u.to(dev), vt.to(dev) @ Q.T
    sign = torch.sign((U * Ue).sum(0))
    err = [float((U - Ue * sign).norm() / Ue.norm()), float((S.cpu() - sv).norm() / sv.norm()),
           float((Vt - Vte * sign[:, None]).norm() / Vte.norm())]
    note(f"[alg2 vectors seed={seed}] " + " ".join(f"{e:.2e}" for e in err))
    # the last directions are eps 2.6e5 = 1.6e-2 off, in U and V^T weighted by what they are of l; four times the largest of
    # twelve inputs of this shape and two others, over two orders of the sums: U 1.2e-4, values 3.1e-7, V^T 4.5e-4
    assert err[0] <= 5e-4 and err[1] <= 1.3e-6 and err[2] <= 1.8e-3, err
