"""Small CG solves as one resident launch (the library's own choice of
execution) against the FP64 oracle and the launch-per-iteration loop.

Sizes and row lengths at the edges of the resident kernel: one row, a
workgroup's rows +- 1, the change from 256 to 512 rows per workgroup, the
most rows a grid holds and one more (which runs the loop), rows that fill the
registers (8 entries), spill to LDS (9, 31) or are too long for one thread
(33).  Tolerances as for the loop (the same arithmetic in the same order
inside a row): FP64 solutions within 1e-12 of the oracle's at tau = 1e-14 and
iteration counts within 1; mixed solutions within 1e-10.  Repeated solves of
one plan, and a solve whose resident launch leaves without a result, are
bitwise equal to what they have to equal."""
import numpy as np
import pytest
import torch

import inputs
import oracle
from tests.gpu_util import DEV, dev_csr, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spk():
    from paper_2510_08230_amd import spk as m
    return m


@pytest.fixture(scope="module")
def ctx(spk):
    c = spk.spk_init(0, torch.cuda.current_stream().cuda_stream)
    yield c
    spk.spk_finalize(c)


@pytest.fixture(autouse=True)
def plain_env(monkeypatch):
    for name in ("SPK_CG_FUSED", "SPK_SPMV_KERNEL", "SPK_RESIDENT"):
        monkeypatch.delenv(name, raising=False)


def band(n, half, seed):
    """Symmetric, strictly dominant, up to 2 half + 1 entries per row, columns ascending."""
    rng = np.random.default_rng(seed)
    up = rng.uniform(-1, 1, (half + 1, n))   # up[d][i] = a(i, i + d)
    cols = np.arange(n)[:, None] + np.arange(-half, half + 1)[None, :]
    inside = (cols >= 0) & (cols < n)
    vals = np.zeros((n, 2 * half + 1))
    for d in range(1, half + 1):
        vals[: n - d, half + d] = up[d][: n - d]
        vals[d:, half - d] = up[d][: n - d]
    vals[:, half] = np.abs(vals).sum(1) + 1.0
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(inside.sum(1), out=rp[1:])
    return inputs.CSR(n, n, rp, cols[inside].astype(np.int32), vals[inside])


def matrix(kind, size, seed):
    if kind == "stencil7":
        return inputs.stencil7(size, seed)
    if kind == "randsym":
        return inputs.randsym(size, seed)
    return band(size, int(kind[4:]), seed)


def config(spk, precision="fp64", tau=1e-14):
    cfg = spk.spk_solver_cfg_default()
    cfg.reduction_factor = tau
    cfg.precision = {"fp64": spk.PREC_FP64, "mixed_fp32": spk.PREC_MIXED_FP32, "mixed_bf16": spk.PREC_MIXED_BF16,
                     "mixed_fp16": spk.PREC_MIXED_FP16}[precision]
    if precision in ("mixed_bf16", "mixed_fp16"):
        cfg.inner_reduction = 1e-2
    return cfg


def solve(spk, ctx, M, bh, cfg, x0=None, times=1):
    pl = spk.spk_plan_solve(ctx, M, cfg)
    out = []
    for _ in range(times):
        x = torch.zeros(M.desc.n_rows, dtype=torch.float64, device=DEV) if x0 is None else to_dev(x0)
        log = spk.spk_execute_solve(pl, to_dev(bh), x)
        out.append((x.cpu().numpy(), log))
    spk.spk_free(pl)
    return out


EDGES = [("band1", 1), ("band1", 2), ("band1", 255), ("band1", 256), ("band1", 257), ("band4", 4097),
         ("band15", 700), ("band16", 700), ("band3", 32768), ("band3", 32769), ("band1", 131072), ("band1", 131073),
         ("stencil7", 17), ("randsym", 1500), ("randsym", 33000)]


@pytest.mark.parametrize("idx", ["i32", "i64"])
@pytest.mark.parametrize("kind,size", EDGES)
def test_fp64_edges(spk, ctx, kind, size, idx):
    A = matrix(kind, size, 3)
    bh = inputs.rhs(A.n_rows, 3)
    runs = solve(spk, ctx, dev_csr(spk, A, ptr=idx, idx=idx), bh, config(spk), times=2)
    xo, ro, _ = oracle.cg(A, bh, tau=1e-14, max_iters=1000)
    x, log = runs[0]
    assert log.stop_reason == spk.STOP_CONVERGED and abs(log.iterations - ro.iterations) <= 1
    assert rel(x, xo) <= 1e-12
    assert log.true_resnorm <= 2e-14 * log.rhs_norm
    assert np.array_equal(x.view(np.uint64), runs[1][0].view(np.uint64)) and runs[1][1].iterations == log.iterations


@pytest.mark.parametrize("precision", ["mixed_fp32", "mixed_bf16", "mixed_fp16"])
@pytest.mark.parametrize("kind,size", [("band1", 257), ("band4", 4097), ("stencil7", 33), ("randsym", 33000)])
def test_mixed(spk, ctx, kind, size, precision):
    A = matrix(kind, size, 5)
    bh = inputs.rhs(A.n_rows, 5)
    (x, log), (x2, log2) = solve(spk, ctx, dev_csr(spk, A), bh, config(spk, precision, 1e-12), times=2)
    xo, _, _ = oracle.cg(A, bh, tau=1e-14, max_iters=1000)
    assert log.stop_reason == spk.STOP_CONVERGED and log.true_resnorm <= 1e-12 * log.rhs_norm
    assert rel(x, xo) <= 1e-10
    assert np.array_equal(x.view(np.uint64), x2.view(np.uint64)) and log2.iterations == log.iterations


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
def test_refused_launch_runs_the_loop(spk, ctx, monkeypatch, precision):
    A = inputs.stencil7(20, 1)
    bh = inputs.rhs(A.n_rows, 1)
    x0 = inputs.vec(A.n_rows, 1, 9)
    M = dev_csr(spk, A)
    cfg = config(spk, precision, 1e-12)
    monkeypatch.setenv("SPK_RESIDENT", "0")
    loop = solve(spk, ctx, M, bh, cfg, x0)[0]
    monkeypatch.setenv("SPK_RESIDENT", "refuse")
    refused = solve(spk, ctx, M, bh, cfg, x0, times=2)
    for x, log in refused:
        assert np.array_equal(x.view(np.uint64), loop[0].view(np.uint64)) and log.iterations == loop[1].iterations
    # a plan whose earlier launches were refused still solves in one launch
    pl = spk.spk_plan_solve(ctx, M, cfg)
    for mode in ("refuse", "1", "1", "refuse", "1"):
        monkeypatch.setenv("SPK_RESIDENT", mode)
        x = to_dev(x0)
        log = spk.spk_execute_solve(pl, to_dev(bh), x)
        assert log.stop_reason == spk.STOP_CONVERGED and rel(x.cpu().numpy(), loop[0]) <= 1e-10
    spk.spk_free(pl)


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
def test_stops(spk, ctx, monkeypatch, precision):
    """Caps, a zero right-hand side, an exact guess, a breakdown and non-finite data stop as in the loop."""
    A = band(600, 5, 2)
    bh = inputs.rhs(600, 2)
    bad = bh.copy()
    bad[3] = np.inf
    neg = inputs.CSR(600, 600, A.row_ptr, A.col, -A.val)
    x0 = inputs.vec(600, 2, 9)
    for M, b, guess, cap in [(A, bh, x0, 0), (A, bh, x0, 1), (A, bh, x0, 7), (A, np.zeros(600), x0, 50),
                             (A, bad, x0, 50), (neg, bh, np.zeros(600), 50), (A, A.val[0] * 0 + bh, x0, 1000)]:
        cfg = config(spk, precision, 1e-12)
        cfg.max_iters = cap
        d = dev_csr(spk, M)
        monkeypatch.setenv("SPK_RESIDENT", "0")
        xl, ll = solve(spk, ctx, d, b, cfg, guess)[0]
        monkeypatch.setenv("SPK_RESIDENT", "1")
        xr, lr = solve(spk, ctx, d, b, cfg, guess)[0]
        assert lr.stop_reason == ll.stop_reason and lr.iterations == ll.iterations
        assert lr.outer_iterations == ll.outer_iterations
        assert np.array_equal(np.isfinite(xr), np.isfinite(xl))
        if np.all(np.isfinite(xl)):
            assert rel(xr, xl) <= 1e-12 if np.any(xl) else not np.any(xr)
