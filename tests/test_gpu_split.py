"""Products whose gathers run ahead in column order (SPK_SPLIT, the kernel
option split=1) against the plain row tiles: the sums run in the same order
on the same values, so products agree bit for bit, and solves agree to the
rounding of their reductions.

Patterns at the edges: blocks gathered from LDS and from L2 (by size and
value type), one block, a ragged last block and tile, empty rows, rectangular
matrices, tiles past the LDS stage and hub rows (which gather for themselves),
64-bit indices, unaligned arrays (which take neither)."""
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


def ragged(n_rows, n_cols, longest, seed):
    """Rows of 0..longest entries at random columns (duplicates allowed, any order)."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, longest + 1, n_rows)
    rp = np.zeros(n_rows + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    nnz = int(rp[-1])
    return inputs.CSR(n_rows, n_cols, rp, rng.integers(0, n_cols, nnz).astype(np.int32), rng.uniform(-1, 1, nnz))


MATS = {
    "randsym_1000": lambda: inputs.randsym(1000, 1),
    "randsym_40000": lambda: inputs.randsym(40000, 2),
    "hubs_60000": lambda: inputs.powerlaw(60000, 3),
    "ragged": lambda: ragged(3001, 50001, 14, 4),
    "wide": lambda: ragged(700, 2200001, 14, 5),          # 135 blocks of 2^14 columns
    "wider": lambda: ragged(700, 16800001, 14, 7),        # 1,026 of them: past the FP64 LDS blocks
    "dense_tiles": lambda: ragged(1500, 20000, 40, 6),    # most tiles past 2,048 entries
    "one_row": lambda: ragged(1, 10, 9, 9),
}


def product(spk, ctx, A, val, idx, kernel, monkeypatch):
    monkeypatch.setenv("SPK_SPLIT", "1")
    monkeypatch.setenv("SPK_COL_CODES", "0")
    monkeypatch.setenv("SPK_SPMV_KERNEL", kernel)
    vt = torch.float64 if val == torch.float64 else torch.float32
    pl = spk.spk_plan_spmv(ctx, dev_csr(spk, A, idx, idx, val))
    x = to_dev(inputs.vec(A.n_cols, 1, 5), vt)
    y = torch.full((A.n_rows,), float("nan"), dtype=vt, device=DEV)
    for _ in range(2):
        spk.spk_execute_spmv(pl, x, y)
    spk.spk_free(pl)
    return y


@pytest.mark.parametrize("name", sorted(MATS))
@pytest.mark.parametrize("val", [torch.float64, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("idx", ["i32", "i64"])
def test_products_bit_equal(spk, ctx, monkeypatch, name, val, idx):
    A = MATS[name]()
    plain = product(spk, ctx, A, val, idx, "stream,remap=64", monkeypatch)
    for opts in ("nt=1,remap=64", "nt=0,remap=0,bpc=16"):
        split = product(spk, ctx, A, val, idx, "stream,split=1," + opts, monkeypatch)
        assert torch.equal(split, plain)


@pytest.mark.parametrize("solver,precision", [("cg", "fp64"), ("cg", "mixed_fp32"), ("cgs", "fp64"), ("gmres", "fp64"),
                                              ("gmres", "mixed_fp16"), ("pcg", "fp64")])
def test_solves(spk, ctx, monkeypatch, solver, precision):
    A = inputs.randsym(150000, 2)
    bh = inputs.rhs(A.n_rows, 2)
    cfg = spk.spk_solver_cfg_default()
    cfg.solver = {"cg": spk.SOLVER_CG, "pcg": spk.SOLVER_CG, "cgs": spk.SOLVER_CGS, "gmres": spk.SOLVER_GMRES}[solver]
    cfg.precond = spk.PRECOND_JACOBI if solver == "pcg" else spk.PRECOND_NONE
    cfg.precision = {"fp64": spk.PREC_FP64, "mixed_fp32": spk.PREC_MIXED_FP32,
                     "mixed_fp16": spk.PREC_MIXED_FP16}[precision]
    cfg.reduction_factor = 1e-12
    monkeypatch.setenv("SPK_SPLIT", "1")
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream,split=1,remap=64,nt=1")
    pl = spk.spk_plan_solve(ctx, dev_csr(spk, A), cfg)
    out = []
    for _ in range(2):
        x = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
        log = spk.spk_execute_solve(pl, to_dev(bh), x)
        assert log.stop_reason == spk.STOP_CONVERGED
        out.append(x.cpu().numpy())
    spk.spk_free(pl)
    xo, _, _ = oracle.cg(A, bh, tau=1e-14, max_iters=1000)
    # kappa <= 18.3 (Gershgorin) and tau = 1e-12
    assert rel(out[0], xo) <= 1e-10
    assert np.array_equal(out[0].view(np.uint64), out[1].view(np.uint64))


def test_solve_of_fp32_values(spk, ctx, monkeypatch):
    """FP32 values: FP32 vectors in the inner loop, FP64 ones in the outer
    residuals; the blocks of one plan serve both."""
    A = inputs.randsym(150000, 2)
    A = inputs.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col, A.val.astype(np.float32).astype(np.float64))
    bh = inputs.rhs(A.n_rows, 2)
    cfg = spk.spk_solver_cfg_default()
    cfg.solver = spk.SOLVER_CG
    cfg.precision = spk.PREC_MIXED_FP32
    cfg.reduction_factor = 1e-12
    monkeypatch.setenv("SPK_SPLIT", "1")
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream,split=1,remap=64,nt=1")
    pl = spk.spk_plan_solve(ctx, dev_csr(spk, A, val=torch.float32), cfg)
    x = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    log = spk.spk_execute_solve(pl, to_dev(bh), x)
    spk.spk_free(pl)
    assert log.stop_reason == spk.STOP_CONVERGED
    xo, _, _ = oracle.cg(A, bh, tau=1e-14, max_iters=1000)
    # kappa <= 18.3 (Gershgorin) and tau = 1e-12
    assert rel(x.cpu().numpy(), xo) <= 1e-10


def test_unaligned_values(spk, ctx, monkeypatch):
    """Values at an odd element: the plan keeps the plain product."""
    monkeypatch.setenv("SPK_SPLIT", "1")
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream,split=1")
    A = inputs.randsym(5000, 1)
    M = dev_csr(spk, A, "i32", "i32")
    buf = torch.empty(A.nnz + 1, dtype=torch.float64, device=DEV)
    buf[1:] = M.tensors[2]
    M2 = spk.CsrMatrix(M.tensors[0], M.tensors[1], buf[1:], A.n_rows, A.n_cols)
    x = to_dev(inputs.vec(A.n_cols, 1, 5))
    y = torch.empty(A.n_rows, dtype=torch.float64, device=DEV)
    pl = spk.spk_plan_spmv(ctx, M2)
    spk.spk_execute_spmv(pl, x, y)
    spk.spk_free(pl)
    assert torch.equal(y, product(spk, ctx, A, torch.float64, "i32", "stream", monkeypatch))
