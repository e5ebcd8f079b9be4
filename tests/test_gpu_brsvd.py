"""End-to-end parity of brsvd_run against the fp64 oracle on the same seeded A and Omega."""
import numpy as np
import pytest
import torch

import paper_1706_07191_amd as B
from paper_1706_07191_amd import synth
from tests.gpu_util import (check_against_oracle, check_full_size_against_oracle, need_gpu, recon_error_fp64_gpu)

pytestmark = pytest.mark.gpu


def _run(cfg, A_dev, Om_dev, row_block=None, a_location=B.BRSVD_A_DEVICE, budget=0, orth=B.BRSVD_ORTH_AUTO,
         pass_mode=B.BRSVD_PASSES_SEPARATE):
    m, n = cfg.m, cfg.n
    prm = B.make_params(m, n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block if row_block is None else row_block,
                        a_location=a_location, device_budget_bytes=budget, orth_method=orth, pass_mode=pass_mode)
    h = B.brsvd_create(prm)
    try:
        U, S, Vt, st = B.brsvd_run(h, A_dev, Om_dev)
        torch.cuda.synchronize()
    finally:
        B.brsvd_destroy(h)
    return U, S, Vt, st


def test_config1_tiny_in_core():
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"]
    A = cfg.make_A()
    Om = cfg.make_Omega()
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    assert st["passes_over_A"] == 2 * cfg.q + 2
    assert st["bytes_A_streamed"] == st["passes_over_A"] * 4 * cfg.m * cfg.n
    assert st["n_blocks"] == 4 and st["orth_fallbacks"] == 0
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, cfg.row_block, U, S, Vt, "C1")


@pytest.mark.parametrize("name,m,n,b", [("C2", 3000, 2500, 700), ("C3", 4000, 3000, 1024), ("C4", 3000, 3500, 900),
                                         ("C1", 333, 271, 100)])
def test_scaled_configs_in_core(name, m, n, b):
    """The recipes of the larger configurations at sizes the oracle finishes in seconds: several
    row blocks with a ragged tail, full sketch widths (l = 110, 272, 144, 30)."""
    dev = need_gpu()
    cfg = synth.CONFIGS[name].scaled(m, n, b)
    print(f"[case] {cfg.name} l={cfg.l} q={cfg.q} b={b}", flush=True)
    A = cfg.make_A()
    Om = cfg.make_Omega()
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, b, U, S, Vt, cfg.name)


def test_largest_sketch_width():
    """l = k + p = 512, the largest width the library accepts, on a matrix barely larger than l."""
    dev = need_gpu()
    m, n, k, p, q, b = 1400, 900, 480, 32, 1, 512
    sig = torch.exp(-torch.arange(600, dtype=torch.float64) / 150.0)
    A = synth.lowrank_plus_noise(m, n, sig, 1e-5, 4242)
    Om = synth.gaussian(n, k + p, 4243)
    cfg = synth.Config("wide", m, n, k, p, q, b, 600, lambda i: i, 1e-5, 4242)
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    check_against_oracle(A.numpy(), Om.numpy(), k, p, q, b, U, S, Vt, "l512")
    with pytest.raises(B.BrsvdError):
        B.brsvd_create(B.make_params(m, n, 500, 13, q))        # l = 513


@pytest.mark.parametrize("m,n,k,p,q,b", [(900, 700, 20, 10, 0, 256),      # no power iteration: sketch and projection only
                                          (640, 64, 8, 8, 3, 640),        # one block, l = 16 = a single column tile, q = 3
                                          (70, 4000, 30, 10, 1, 32),      # very wide: fewer rows than a row tile per block
                                          (4100, 33, 5, 0, 2, 1000),      # p = 0, odd n (rows at every alignment), ragged tail of 100 rows
                                          (50, 40, 39, 1, 1, 7)])         # l = min(m, n): the sketch spans everything
def test_degenerate_shapes_and_parameters(m, n, k, p, q, b):
    dev = need_gpu()
    sig = 0.9 ** torch.arange(min(m, n), dtype=torch.float64)
    A = synth.lowrank_plus_noise(m, n, sig, 1e-3, 5150 + m)
    Om = synth.gaussian(n, k + p, 5151 + n)
    cfg = synth.Config("edge", m, n, k, p, q, b, min(m, n), lambda i: i, 1e-3, 5150)
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    assert st["passes_over_A"] == 2 * q + 2 and st["n_blocks"] == -(-m // b)
    check_against_oracle(A.numpy(), Om.numpy(), k, p, q, b, U, S, Vt, f"edge {m}x{n} l={k + p} q={q}")


def test_seeded_random_shapes_against_oracle():
    """Forty seeded random problems (shape, rank parameters, block size, pass mode, storage): every one within the
    usual tolerances of the oracle.  Exercises ragged tiles, single-row blocks and the launch plans of odd shapes."""
    import random
    dev = need_gpu()
    rng = random.Random(17060719)
    for case in range(40):
        m = rng.choice([rng.randint(40, 400), rng.randint(400, 3000)])
        n = rng.choice([rng.randint(40, 400), rng.randint(400, 3000)])
        l = rng.randint(2, min(m, n, 61) - 1)        # sigma_l / sigma_1 >= 0.96^60 = 0.09: resolved in fp32 in either pass mode
        p = rng.randint(0, min(l - 1, 12))
        k = l - p
        q = rng.randint(0, 3)
        b = rng.choice([0, rng.randint(1, m), rng.randint(max(1, m // 8), m)])
        fused = rng.random() < 0.3
        host = rng.random() < 0.25
        sig = torch.tensor([0.96 ** i for i in range(min(m, n))], dtype=torch.float64)
        A = synth.lowrank_plus_noise(m, n, sig, 1e-3, 9000 + case)
        Om = synth.gaussian(n, l, 9500 + case)
        cfg = synth.Config(f"rand{case}", m, n, k, p, q, b, min(m, n), lambda i: i, 1e-3, 9000 + case)
        print(f"[case {case}] m={m} n={n} k={k} p={p} q={q} b={b} fused={fused} host={host}", flush=True)
        U, S, Vt, st = _run(cfg, A.pin_memory() if host else A.to(dev), Om.to(dev),
                            a_location=B.BRSVD_A_HOST_PINNED if host else B.BRSVD_A_DEVICE,
                            pass_mode=B.BRSVD_PASSES_FUSED if fused else B.BRSVD_PASSES_SEPARATE)
        assert st["fused_fallbacks"] == 0                # sigma_l / sigma_1 >= 0.09: far above the fused mode's floor
        assert st["passes_over_A"] == (q + 1 if fused and host else 2 * q + 2) * (1 + st["orth_fallbacks"])
        assert st["bytes_A_read_by_kernels"] == (2 * q + 2) * (1 + st["orth_fallbacks"]) * 4 * m * n
        check_against_oracle(A.numpy(), Om.numpy(), k, p, q, b if b else m, U, S, Vt, f"rand{case}")


def test_zero_and_nonfinite_inputs_end_with_a_status():
    """A = 0 has no range to orthonormalise: every route reports the breakdown as a status (no hang, no
    crash); the handle stays usable.  NaN input: the call returns (values unspecified)."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"].scaled(600, 400, 256)
    Om = cfg.make_Omega().to(dev)
    h = B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=256))
    try:
        with pytest.raises(B.BrsvdError) as ei:
            B.brsvd_run(h, torch.zeros(cfg.m, cfg.n, device=dev), Om)
        assert ei.value.status == B.BRSVD_ERR_ORTH_BREAKDOWN
        A = cfg.make_A().to(dev)
        U, S, Vt, st = B.brsvd_run(h, A, Om)                      # the same handle afterwards
        check_against_oracle(A.cpu().numpy(), Om.cpu().numpy(), cfg.k, cfg.p, cfg.q, 256, U, S, Vt, "after-zero")
        An = A.clone()
        An[17, 23] = float("nan")
        try:
            B.brsvd_run(h, An, Om)
        except B.BrsvdError:
            pass
        U2, S2, Vt2, _ = B.brsvd_run(h, A, Om)
        assert torch.equal(S, S2)
    finally:
        B.brsvd_destroy(h)


def test_caller_streams():
    """Caller-owned compute and copy streams (default priority): in-core on a side stream, and host-resident A
    with both streams supplied; results equal the default-stream runs bit for bit."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"]
    A, Om = cfg.make_A(), cfg.make_Omega()
    Ad, Od = A.to(dev), Om.to(dev)
    U0, S0, Vt0, _ = _run(cfg, Ad, Od)
    cs, ps = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    h = B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block, compute_stream=cs))
    try:
        U1, S1, Vt1, st1 = B.brsvd_run(h, Ad, Od)
    finally:
        B.brsvd_destroy(h)
    assert torch.equal(S0, S1) and torch.equal(U0, U1) and torch.equal(Vt0, Vt1) and st1["total_seconds"] > 0
    Ah = A.pin_memory()
    outs = []
    for kw in (dict(), dict(compute_stream=cs, copy_stream=ps)):
        h = B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block,
                                         a_location=B.BRSVD_A_HOST_PINNED, **kw))
        try:
            outs.append(B.brsvd_run(h, Ah, Od))
        finally:
            B.brsvd_destroy(h)
    torch.cuda.synchronize()
    assert torch.equal(outs[0][1], outs[1][1]) and torch.equal(outs[0][0], outs[1][0])
    assert outs[1][3]["copy_seconds"] > 0 and outs[1][3]["n_blocks"] == 4


def test_caller_owned_workspace():
    """A handle built on a device buffer of the caller (no allocation in brsvd_create) gives the same results bit
    for bit as one that allocates its own; too small a buffer is refused; the buffer survives brsvd_destroy."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"]
    A, Om = cfg.make_A(), cfg.make_Omega()
    Ad, Od = A.to(dev), Om.to(dev)
    U0, S0, Vt0, _ = _run(cfg, Ad, Od)
    for host in (False, True):
        loc = B.BRSVD_A_HOST_PINNED if host else B.BRSVD_A_DEVICE
        need = B.brsvd_workspace_bytes(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block, a_location=loc))
        ws = torch.empty(need + 4096, dtype=torch.uint8, device=dev)
        ws.fill_(0xAB)                                  # whatever the buffer held before must not matter
        h = B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block, a_location=loc,
                                         workspace=ws))
        try:
            U1, S1, Vt1, st = B.brsvd_run(h, A.pin_memory() if host else Ad, Od)
        finally:
            B.brsvd_destroy(h)
        torch.cuda.synchronize()
        assert torch.all(ws[need:] == 0xAB)             # nothing written beyond the declared working set
        if host:
            rel = ((S1[:cfg.k] - S0[:cfg.k]).abs() / S0[:cfg.k]).max().item()
            assert rel < 2e-5                           # block-wise launches sum in another order than one launch
        else:
            assert torch.equal(S0, S1) and torch.equal(U0, U1) and torch.equal(Vt0, Vt1)
        check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, cfg.row_block, U1, S1, Vt1, f"workspace host={host}")
        with pytest.raises(B.BrsvdError) as ei:
            B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block, a_location=loc,
                                         workspace=ws[:need - 256]))
        assert ei.value.status == B.BRSVD_ERR_BUDGET


@pytest.mark.parametrize("host", [False, True])
def test_a_workspace_in_host_memory_is_refused(host):
    """brsvd_create clears a few bytes of the workspace, which the runtime refuses for pageable host memory: no kernel ever sees it."""
    need_gpu()
    par = dict(row_block=400, a_location=B.BRSVD_A_HOST_PINNED if host else B.BRSVD_A_DEVICE)
    need = B.brsvd_workspace_bytes(B.make_params(900, 700, 20, 10, 1, **par))
    ws = torch.zeros(need + 256, dtype=torch.uint8)
    at = -ws.data_ptr() % 256
    with pytest.raises(B.BrsvdError) as ei:
        B.brsvd_create(B.make_params(900, 700, 20, 10, 1, workspace=ws[at:at + need], **par))
    B.lib().hipGetLastError()                        # the runtime's own record of the refused call
    assert ei.value.status == B.BRSVD_ERR_HIP and not bool(ws.any())


@pytest.mark.parametrize("m,n,k,p", [(900, 700, 20, 10), (1200, 900, 100, 10), (1300, 1100, 256, 16), (5000, 60, 16, 4)])
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("method", [B.BRSVD_ORTH_AUTO, B.BRSVD_ORTH_TSQR])
def test_nothing_in_the_workspace_has_to_be_cleared(m, n, k, p, f64, method):
    """A workspace that is full of NaN gives the bits of one that is full of zeros: both schemes and a robust-PCA iteration."""
    dev = need_gpu()
    print(f"[case] workspace {m} x {n} l={k + p} f64={f64} method={method}", flush=True)
    dt = torch.float64 if f64 else torch.float32
    A = synth.gaussian(m, n, 61, dtype=dt).to(dev)
    Om = synth.gaussian(n, k + p, 62, dtype=dt).to(dev)
    out = []
    for fill in (0x00, 0xff):
        par = dict(row_block=400, orth_method=method, dtype=B.BRSVD_DTYPE_F64 if f64 else B.BRSVD_DTYPE_F32)
        need = B.brsvd_workspace_bytes(B.make_params(m, n, k, p, 1, **par))
        res = []
        for call in ("run", "alg2", "rpca"):
            ws = torch.full((need,), fill, dtype=torch.uint8, device=dev)
            h = B.brsvd_create(B.make_params(m, n, k, p, 1, workspace=ws, **par))
            try:
                if call == "run":
                    res += B.brsvd_run(h, A, Om)[:3]
                elif call == "alg2":
                    res += B.brsvd_run_alg2(h, A, k + p, seed=5)[:3]
                else:
                    res += B.brsvd_rpca_ialm_tol(h, A, Om.reshape(1, n, k + p), 1, 0.0, 0.05, 0.02, 1.5, norm2_M=80.0)[:2]
            finally:
                B.brsvd_destroy(h)
        out.append(res)
    assert all(torch.equal(a, b) and bool(torch.isfinite(a).all()) for a, b in zip(*out))


@pytest.mark.parametrize("m,n,l,block", [(8199, 187, 184, 8025), (9056, 274, 185, 4022)])
def test_row_block_changes_no_bit_of_a_resident_svd(m, n, l, block):
    """A in device memory is not walked in blocks by brsvd_run, so the row block may not show in the result.  These are sizes where the scratch of
    that block's products has room for one more piece of a panel's product with an l x l factor than the scratch of A's own."""
    dev = need_gpu()
    print(f"[case] row blocks {m} x {n} l={l}", flush=True)
    A = synth.gaussian(m, n, 71).to(dev)
    Om = synth.gaussian(n, l, 72).to(dev)
    out = []
    for b in (512, block, m):
        h = B.brsvd_create(B.make_params(m, n, l - 3, 3, 1, row_block=b))
        try:
            out.append(B.brsvd_run(h, A, Om)[:3])
        finally:
            B.brsvd_destroy(h)
    for other in out[1:]:
        assert all(torch.equal(x, y) for x, y in zip(out[0], other))


def test_timing_levels():
    """timing_level 1 times the pass kernels and the whole call only; the results do not depend on it."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"]
    A, Om = cfg.make_A().to(dev), cfg.make_Omega().to(dev)
    out = {}
    for level in (0, 1):
        h = B.brsvd_create(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block, timing_level=level))
        try:
            out[level] = B.brsvd_run(h, A, Om)
        finally:
            B.brsvd_destroy(h)
    s0, s1 = out[0][3], out[1][3]
    assert s0["orth_seconds"] > 0 and s0["svd_seconds"] > 0 and s0["lift_seconds"] > 0
    assert s1["orth_seconds"] == 0 and s1["svd_seconds"] == 0 and s1["lift_seconds"] == 0
    for s in (s0, s1):
        assert s["gemm_an_seconds"] > 0 and s["gemm_at_seconds"] > 0
        assert s["total_seconds"] >= s["gemm_an_seconds"] + s["gemm_at_seconds"]
        assert s["gemm_an_launches"] == 3 and s["gemm_at_launches"] == 3
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0], out[1][0])


def test_forced_tsqr_matches_oracle():
    dev = need_gpu()
    cfg = synth.CONFIGS["C2"].scaled(3000, 2500, 700)
    A = cfg.make_A()
    Om = cfg.make_Omega()
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev), orth=B.BRSVD_ORTH_TSQR)
    assert st["orth_fallbacks"] == 0
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, 700, U, S, Vt, "C2-tsqr")


@pytest.mark.parametrize("name,m,n,b,q", [("C2", 3000, 2500, 700, 2), ("C3", 4000, 3000, 1024, 1),
                                           ("C1", 2000, 1000, 512, 2), ("C1", 1500, 800, 333, 0)])
def test_fused_passes_match_oracle(name, m, n, b, q):
    """Fused pass mode: both products of a power step without an orthonormalisation in between, projection
    recovered as C^T R^-1.  Same range(Y) in exact arithmetic, so the same oracle applies."""
    dev = need_gpu()
    cfg = synth.CONFIGS[name].scaled(m, n, b)
    cfg.q = q
    A = cfg.make_A()
    Om = cfg.make_Omega()
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev), pass_mode=B.BRSVD_PASSES_FUSED)
    # A lives in device memory here: each of the two product kernels of a fused pass reads it, and that is what
    # the statistics count; only a host-resident A is read q+1 times (over the host link)
    assert st["passes_over_A"] == 2 * q + 2 and st["bytes_A_streamed"] == (2 * q + 2) * 4 * m * n
    assert st["gemm_an_launches"] == q + 1 and st["gemm_at_launches"] == q + 1
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, q, b, U, S, Vt, f"{cfg.name}-fused-q{q}")


@pytest.mark.parametrize("depth,expect_fallback", [(2e-2, False), (5e-3, False), (1e-3, True), (3e-4, True)])
def test_fused_mode_accuracy_limit_and_guard(depth, expect_fallback):
    """What the fused pass mode guarantees in fp32.  Its projection B^T = C^T R^-1 multiplies the rounding noise of
    C^T by (sigma_1 / sigma_l)^2, so it keeps the 1e-4 tolerance only while sigma_l / sigma_1 stays above about the
    square root of the machine epsilon; past that the unguarded scheme returns trailing values that are wrong by
    factors (measured: 0.5 relative at sigma_k / sigma_1 = 1e-3, 7 at 3e-4), and too LARGE, so they would displace
    real ones.  The library therefore checks the diagonal of the sketch's triangular factor and repeats such a run
    with separate passes.  Pinned here on exactly known geometric spectra from sigma_1 = 1 down to sigma_k = depth
    (tail 0.3 depth 0.9^j): above the floor the fused run stands and meets the tolerance; below it the fallback is
    taken, is counted, and the result meets the tolerance again.  The separate mode meets it throughout."""
    dev = need_gpu()
    m, n, k, p, q, b = 3000, 2000, 40, 10, 1, 1024
    s = torch.cat([torch.logspace(0, np.log10(depth), k, dtype=torch.float64),
                   depth * 0.3 * 0.9 ** torch.arange(1, 61, dtype=torch.float64)])
    A = synth.exact_spectrum_matrix(m, n, s, seed=4711, dtype=torch.float32)
    Om = synth.gaussian(n, k + p, 4712)
    cfg = synth.Config("depth", m, n, k, p, q, b, 100, lambda i: i, 0.0, 4711)
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    assert st["fused_fallbacks"] == 0 and st["passes_over_A"] == 2 * q + 2
    check_against_oracle(A.numpy(), Om.numpy(), k, p, q, b, U, S, Vt, f"depth {depth:g} separate")
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev), pass_mode=B.BRSVD_PASSES_FUSED)
    assert st["fused_fallbacks"] == (1 if expect_fallback else 0)
    assert st["passes_over_A"] == (2 * q + 2) * (2 if expect_fallback else 1)
    check_against_oracle(A.numpy(), Om.numpy(), k, p, q, b, U, S, Vt, f"depth {depth:g} fused")


def test_fused_passes_host_resident_and_tsqr():
    dev = need_gpu()
    cfg = synth.CONFIGS["C4"].scaled(3000, 3500, 900)
    A = cfg.make_A()
    Om = cfg.make_Omega()
    Ap = torch.empty(cfg.m, cfg.n, dtype=torch.float32, pin_memory=True)
    Ap.copy_(A)
    U, S, Vt, st = _run(cfg, Ap, Om.to(dev), a_location=B.BRSVD_A_HOST_PINNED, pass_mode=B.BRSVD_PASSES_FUSED)
    assert st["passes_over_A"] == 2 and st["n_blocks"] == 4 and st["gemm_an_launches"] == 8
    assert st["bytes_A_streamed"] == 2 * 4 * cfg.m * cfg.n and st["bytes_A_read_by_kernels"] == 4 * 4 * cfg.m * cfg.n
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, 900, U, S, Vt, "C4-host-fused")
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev), orth=B.BRSVD_ORTH_TSQR, pass_mode=B.BRSVD_PASSES_FUSED)
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, 900, U, S, Vt, "C4-fused-tsqr")


def test_block_size_independence_and_determinism():
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"]
    A = cfg.make_A().to(dev)
    Om = cfg.make_Omega().to(dev)
    ref = _run(cfg, A, Om)
    again = _run(cfg, A, Om)
    assert torch.equal(ref[1], again[1]) and torch.equal(ref[0], again[0]) and torch.equal(ref[2], again[2])
    for b in (2000, 64, 777):
        out = _run(cfg, A, Om, row_block=b)
        rel = ((out[1][:cfg.k] - ref[1][:cfg.k]).abs() / ref[1][:cfg.k]).max().item()
        assert rel < 2e-5, (b, rel)


def test_host_resident_streaming_matches_in_core():
    """A in pinned host memory, streamed through the two staging buffers (ragged last block)."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C4"].scaled(3000, 3500, 900)
    A = cfg.make_A()
    Om = cfg.make_Omega()
    Ap = torch.empty(cfg.m, cfg.n, dtype=torch.float32, pin_memory=True)
    Ap.copy_(A)
    U, S, Vt, st = _run(cfg, Ap, Om.to(dev), a_location=B.BRSVD_A_HOST_PINNED)
    assert st["n_blocks"] == 4 and st["gemm_an_launches"] == 4 * (cfg.q + 1)
    check_against_oracle(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, 900, U, S, Vt, "C4-host")
    # budget-driven block size: working set must respect the cap
    need = B.brsvd_workspace_bytes(B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=256,
                                                 a_location=B.BRSVD_A_HOST_PINNED))
    U2, S2, Vt2, st2 = _run(cfg, Ap, Om.to(dev), row_block=0, a_location=B.BRSVD_A_HOST_PINNED, budget=need + (8 << 20))
    assert 256 <= st2["row_block"] < cfg.m
    rel = ((S2[:cfg.k] - S[:cfg.k]).abs() / S[:cfg.k]).max().item()
    assert rel < 2e-5


def test_exact_rank_input_fp32_error_level():
    """Exactly rank-r input, r <= k: the paper reports ~1e-7 relative error in single precision."""
    dev = need_gpu()
    r, k, p = 12, 16, 8
    s = torch.linspace(10.0, 1.0, r, dtype=torch.float64)
    A = synth.exact_spectrum_matrix(1500, 900, s, seed=77, dtype=torch.float32)
    Om = synth.gaussian(900, k + p, 78)
    cfg = synth.Config("rank", 1500, 900, k, p, 1, 400, r, lambda i: i, 0.0, 0)
    U, S, Vt, st = _run(cfg, A.to(dev), Om.to(dev))
    # rank r < l: the sketch panels are numerically rank deficient; the clamped first CholeskyQR sweep
    # normally copes (no rerun), the Householder-tree rerun remains the fallback
    assert st["orth_fallbacks"] in (0, 1) and st["passes_over_A"] == (1 + st["orth_fallbacks"]) * (2 * cfg.q + 2)
    sg = S.double().cpu().numpy()
    assert np.max(np.abs(sg[:r] - s.numpy()) / s.numpy()) < 1e-5
    assert np.all(sg[r:] < 1e-5 * sg[0])
    from oracle import brsvd_oracle as O
    err = O.recon_error(A.numpy(), U.double().cpu().numpy(), sg, Vt.double().cpu().numpy())
    assert err < 2e-6
    # U to the usual bound; the right vectors of the l - r noise triplets (sigma ~ 1e-8 sigma_1) are only
    # determined to ~1e-5, on either orthonormalisation route; the r meaningful ones to the usual bound
    Vn = Vt.double().cpu().numpy().T
    assert O.orth_defect(U.double().cpu().numpy()) <= 1e-5
    assert O.orth_defect(Vn[:, :r]) <= 1e-5 and O.orth_defect(Vn) <= 1e-4
    # forced Householder-tree route on the same input
    U2, S2, Vt2, st2 = _run(cfg, A.to(dev), Om.to(dev), orth=B.BRSVD_ORTH_TSQR)
    assert np.max(np.abs(S2.double().cpu().numpy()[:r] - s.numpy()) / s.numpy()) < 1e-5
    assert O.orth_defect(U2.double().cpu().numpy()) <= 1e-5


# ---- full-size configurations, in the launch configuration bench.py times ---------------------------

def _fp64_properties(A_rows, m, n, U, S, Vt, dev, step=4096):
    """Checks that hold at any size, evaluated in fp64 on the GPU block by block (checker only):
    orthogonality of U and V, the triplet identity U^T A = diag(S) V^T, and the rank-l error through
    ||A - U S V^T||_F^2 = ||A||_F^2 - sum S^2.  A_rows(r0, r1) returns rows of A as a CUDA tensor."""
    l = S.numel()
    Ud, Vd, Sd = U.double(), Vt.double(), S.double()
    eye = torch.eye(l, device=dev, dtype=torch.float64)
    orthU = torch.linalg.matrix_norm(Ud.T @ Ud - eye, 2).item()
    orthV = torch.linalg.matrix_norm(Vd @ Vd.T - eye, 2).item()
    acc = torch.zeros(l, n, device=dev, dtype=torch.float64)
    nA2 = 0.0
    for r0 in range(0, m, step):
        blk = A_rows(r0, min(m, r0 + step)).double()
        acc += Ud[r0:r0 + step].T @ blk
        nA2 += float((blk * blk).sum())
    triplet = torch.linalg.matrix_norm(acc - Sd[:, None] * Vd).item() / float(Sd[0])
    err_l = float(np.sqrt(max(nA2 - float((Sd ** 2).sum()), 0.0) / nA2))
    return orthU, orthV, triplet, err_l


def test_config2_full_size_against_oracle():
    """The benchmark workload itself: 20000 x 20000, k=100, p=10, q=2, row block 4096 (oracle: ~3 s)."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C2"]
    A = cfg.make_A(device=dev)
    Om = cfg.make_Omega(device=dev)
    U, S, Vt, st = _run(cfg, A, Om)
    assert st["n_blocks"] == 5 and st["passes_over_A"] == 6
    check_against_oracle(A.cpu().numpy(), Om.cpu().numpy(), cfg.k, cfg.p, cfg.q, cfg.row_block, U, S, Vt, "C2-full")


def test_fp64_gpu_checker_equals_oracle_metric():
    """The block-wise fp64 reconstruction error evaluated on the GPU (used as the checker at the large sizes) is the
    oracle's recon_error: same numbers on a case both can evaluate."""
    from oracle import brsvd_oracle as O
    dev = need_gpu()
    cfg = synth.CONFIGS["C1"].scaled(1300, 700, 512)
    A, Om = cfg.make_A(), cfg.make_Omega()
    Uo, so, Vto = O.brsvd(A.numpy(), Om.numpy(), cfg.k, cfg.p, cfg.q, row_block=512)
    Ad = A.to(dev)
    for k in (cfg.k, None, 3):
        ref = O.recon_error(A.numpy(), Uo, so, Vto, k=k)
        got = recon_error_fp64_gpu(lambda a, b: Ad[a:b], cfg.m, Uo, so, Vto, k=k, step=500)
        assert abs(got - ref) <= 1e-12 * ref


def test_config3_full_size_against_oracle():
    """100000 x 50000 (20 GB), k=256, p=16, q=1, row block 8192, in the launch configuration bench.py times, against
    the complete fp64 oracle walked over the same matrix (about half a minute of host time on 16 cores)."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C3"]
    free, _ = torch.cuda.mem_get_info()
    if free < 40 * 2 ** 30:
        pytest.skip("needs 40 GB of free HBM")
    A = cfg.make_A(device=dev)
    Om = cfg.make_Omega(device=dev)
    U, S, Vt, st = _run(cfg, A, Om)
    assert st["n_blocks"] == 13 and st["passes_over_A"] == 4 and st["orth_fallbacks"] == 0
    orthU, orthV, triplet, err_l = _fp64_properties(lambda a, b: A[a:b], cfg.m, cfg.n, U, S, Vt, dev)
    print(f"[C3-full] orthU={orthU:.2e} orthV={orthV:.2e} triplet={triplet:.2e} err_l={err_l:.4e}", flush=True)
    assert orthU <= 1e-5 and orthV <= 1e-5 and triplet <= 1e-4
    # sampled rows of the sketch pass against the oracle's definition Y[i,:] = A[i,:] Omega
    rows = torch.tensor([0, 1, 8191, 8192, 50000, 98303, 99999], device=dev)
    Y = B.brsvd_gemm_an(A, Om)
    ref = A[rows].double().cpu().numpy() @ Om.double().cpu().numpy()
    got = Y[rows].double().cpu().numpy()
    assert np.max(np.abs(got - ref)) <= 1e-4 * np.max(np.abs(ref))
    del Y
    check_full_size_against_oracle(A.cpu().numpy(), lambda a, b: A[a:b], Om.cpu().numpy(), cfg, U, S, Vt, "C3-full")


def test_config4_streaming_large_block_against_oracle():
    """The out-of-core recipe at its real column count and row block (16384 x 100000 blocks, 16 GB budget) with
    40000 rows (16 GB pinned: three blocks, ragged tail), against the complete fp64 oracle walked over the same
    pinned buffer.  (The GPU machine caps pinned host memory at about 64 GB, so the 80 GB matrix itself cannot be
    allocated there; bench.py times the recipe at 160000 rows.)"""
    dev = need_gpu()
    cfg = synth.CONFIGS["C4"].scaled(40000, 100000)
    pm = B.PinnedMatrix(cfg.m, cfg.n)
    try:
        cfg.make_A(device="cpu", out=pm.tensor, gen_device=dev)
        Om = cfg.make_Omega(device=dev)
        prm = B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block,
                            a_location=B.BRSVD_A_HOST_PINNED, device_budget_bytes=cfg.device_budget)
        assert B.brsvd_workspace_bytes(prm) <= cfg.device_budget
        h = B.brsvd_create(prm)
        try:
            U, S, Vt, st = B.brsvd_run(h, pm.tensor, Om, pinned=True)
        finally:
            B.brsvd_destroy(h)
        assert st["n_blocks"] == 3 and st["gemm_an_launches"] == 6 and st["copy_seconds"] > 0
        assert st["passes_over_A"] == 4 and st["bytes_A_streamed"] == 4 * 4 * cfg.m * cfg.n
        A_rows = lambda a, b: pm.tensor[a:b].to(dev)
        orthU, orthV, triplet, err_l = _fp64_properties(A_rows, cfg.m, cfg.n, U, S, Vt, dev)
        print(f"[C4-40000] orthU={orthU:.2e} orthV={orthV:.2e} triplet={triplet:.2e} err_l={err_l:.4e} "
              f"link={st['bytes_A_streamed'] / st['total_seconds'] / 1e9:.1f} GB/s", flush=True)
        assert orthU <= 1e-5 and orthV <= 1e-5 and triplet <= 1e-4
        check_full_size_against_oracle(pm.tensor.numpy(), A_rows, Om.cpu().numpy(), cfg, U, S, Vt, "C4-40000x100000")
        # the same matrix resident in HBM gives the same singular values
        A_dev = pm.tensor.to(dev)
        U2, S2, Vt2, _ = _run(cfg, A_dev, Om)
        rel = ((S2[:cfg.k] - S[:cfg.k]).abs() / S[:cfg.k]).max().item()
        assert rel < 2e-5
    finally:
        pm.free()


def test_config4_at_the_largest_pinnable_size_properties():
    """The out-of-core configuration at 160000 of its 200000 rows (64 GB of pinned host memory, what the GPU machine lets a
    process pin; bench.py times this size): ten blocks of 16384 x 100000 through two staging buffers under the 16 GiB
    device budget.  The oracle takes minutes at this size, so the result is held to what holds at any size, evaluated
    in fp64 on the GPU: orthonormal U and V, the triplet identity U^T A = diag(S) V^T, and sigma against the same
    recipe's resident-in-HBM run."""
    dev = need_gpu()
    cfg = synth.CONFIGS["C4"].scaled(160000, 100000)
    try:
        pm = B.PinnedMatrix(cfg.m, cfg.n)
    except MemoryError as e:                            # a box that pins less: the 40000-row test above still ran
        pytest.skip(f"cannot pin 64 GB on this box: {e}")
    try:
        print("[case] C4 at 160000 rows: generating A", flush=True)
        cfg.make_A(device="cpu", out=pm.tensor, gen_device=dev)
        Om = cfg.make_Omega(device=dev)
        prm = B.make_params(cfg.m, cfg.n, cfg.k, cfg.p, cfg.q, row_block=cfg.row_block,
                            a_location=B.BRSVD_A_HOST_PINNED, device_budget_bytes=cfg.device_budget)
        assert B.brsvd_workspace_bytes(prm) <= cfg.device_budget
        h = B.brsvd_create(prm)
        try:
            print("[case] C4 at 160000 rows: streaming run", flush=True)
            U, S, Vt, st = B.brsvd_run(h, pm.tensor, Om, pinned=True)
        finally:
            B.brsvd_destroy(h)
        assert st["n_blocks"] == 10 and st["passes_over_A"] == 4 and st["bytes_A_streamed"] == 4 * 4 * cfg.m * cfg.n
        A_rows = lambda a, b: pm.tensor[a:b].to(dev)
        print("[case] C4 at 160000 rows: fp64 properties", flush=True)
        orthU, orthV, triplet, err_l = _fp64_properties(A_rows, cfg.m, cfg.n, U, S, Vt, dev)
        print(f"[C4-160000] orthU={orthU:.2e} orthV={orthV:.2e} triplet={triplet:.2e} err_l={err_l:.4e} "
              f"seconds={st['total_seconds']:.3f} link={st['bytes_A_streamed'] / st['total_seconds'] / 1e9:.1f} GB/s", flush=True)
        assert orthU <= 1e-5 and orthV <= 1e-5 and triplet <= 1e-4
        sg = S.double().cpu().numpy()
        assert np.all(np.diff(sg) <= 0) and np.all(sg >= 0)
        # the same 64 GB resident in HBM (288 GB of it): same singular values
        A_dev = torch.empty(cfg.m, cfg.n, device=dev, dtype=torch.float32)
        for r0 in range(0, cfg.m, 16384):
            A_dev[r0:r0 + 16384].copy_(pm.tensor[r0:r0 + 16384], non_blocking=False)
        U2, S2, Vt2, _ = _run(cfg, A_dev, Om)
        rel = ((S2[:cfg.k] - S[:cfg.k]).abs() / S[:cfg.k]).max().item()
        print(f"[C4-160000] sigma host-resident vs device-resident: {rel:.2e}", flush=True)
        assert rel < 2e-5
        del A_dev
    finally:
        pm.free()
