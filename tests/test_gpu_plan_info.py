"""What spk_plan_get_info says of the path a plan takes, at the edges of the
rules: a small CG solve as one resident launch (its rows' length, the entries
that a workgroup keeps, the solver and the switches), and products whose
gathers run ahead.  The solves are checked against the FP64 oracle as the
other resident ones are (solutions within 1e-12 at tau = 1e-14, mixed ones
within 1e-10 at 1e-12)."""
import numpy as np
import pytest
import torch

import inputs
import oracle
from tests.gpu_util import DEV, dev_csr, rel, to_dev
from tests.test_gpu_resident import band
from tests.test_gpu_split import ragged

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
    for name in ("SPK_CG_FUSED", "SPK_SPMV_KERNEL", "SPK_RESIDENT", "SPK_LONG_ROWS", "SPK_SPLIT", "SPK_COL_CODES"):
        monkeypatch.delenv(name, raising=False)


# half, n, resident in FP64, in mixed precision.  Entries past eight per row go to LDS: 36 bytes for every entry of a
# workgroup in FP64 (4,323 fit), 20 in mixed precision (7,782); 256 rows per workgroup up to 32,768, 512 above.
SOLVES = [(3, 131072, True, True), (3, 131073, False, False),
          (4, 300, True, True), (7, 1000, True, True),      # 9 and 15 entries: 2,304 and 3,840 per workgroup
          (8, 1000, False, True),                           # 17: 4,352
          (15, 139, True, True),                            # 31 entries, 4,069 in all
          (15, 256, False, True), (15, 700, False, False),  # 7,696; 7,936 - 120 in the fullest workgroup but one
          (16, 50, False, False),                           # a row of 33
          (4, 32769, False, True), (7, 40000, False, True), (8, 40000, False, False)]


@pytest.mark.parametrize("half,n,fp64,mixed", SOLVES)
def test_resident_solves(spk, ctx, half, n, fp64, mixed):
    A = band(n, half, 3)
    bh = inputs.rhs(n, 3)
    xo, ro, _ = oracle.cg(A, bh, tau=1e-14, max_iters=1000)
    M = dev_csr(spk, A)
    for precision, tau, tol, want in ((spk.PREC_FP64, 1e-14, 1e-12, fp64), (spk.PREC_MIXED_FP32, 1e-12, 1e-10, mixed)):
        cfg = spk.spk_solver_cfg_default()
        cfg.precision, cfg.reduction_factor = precision, tau
        pl = spk.spk_plan_solve(ctx, M, cfg)
        mode = spk.spk_plan_get_info(pl)["exec_mode"]
        x = torch.zeros(n, dtype=torch.float64, device=DEV)
        log = spk.spk_execute_solve(pl, to_dev(bh), x)
        after = spk.spk_plan_get_info(pl)["exec_mode"]
        spk.spk_free(pl)
        assert mode == after == (spk.EXEC_RESIDENT if want else spk.EXEC_HOST_LOOP)
        assert log.stop_reason == spk.STOP_CONVERGED and rel(x.cpu().numpy(), xo) <= tol


def test_other_solves_are_not_resident(spk, ctx, monkeypatch):
    A = inputs.stencil7(8, 1)
    M = dev_csr(spk, A)

    def mode(**fields):
        cfg = spk.spk_solver_cfg_default()
        for k, v in fields.items():
            setattr(cfg, k, v)
        pl = spk.spk_plan_solve(ctx, M, cfg)
        out = spk.spk_plan_get_info(pl)["exec_mode"]
        spk.spk_free(pl)
        return out

    assert mode() == spk.EXEC_RESIDENT
    assert mode(max_iters=100_000) == spk.EXEC_RESIDENT and mode(max_iters=100_001) == spk.EXEC_HOST_LOOP
    assert mode(precond=spk.PRECOND_JACOBI) == spk.EXEC_HOST_LOOP
    assert mode(solver=spk.SOLVER_CGS) == spk.EXEC_HOST_LOOP and mode(solver=spk.SOLVER_GMRES) == spk.EXEC_HOST_LOOP
    for m in (spk.EXEC_HOST_LOOP, spk.EXEC_GRAPH, spk.EXEC_PERSISTENT):
        assert mode(exec_mode=m) == m
    with pytest.raises(spk.SpkError) as e:   # a report, not a choice
        mode(exec_mode=spk.EXEC_RESIDENT)
    assert e.value.status == spk.ERR_INVALID_ARG
    monkeypatch.setenv("SPK_RESIDENT", "0")
    assert mode() == spk.EXEC_HOST_LOOP


def test_a_timeout_shows(spk, ctx, monkeypatch):
    A = inputs.stencil7(8, 1)
    pl = spk.spk_plan_solve(ctx, dev_csr(spk, A), spk.spk_solver_cfg_default())
    x = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    modes = []
    for env in ("refuse", "timeout"):
        monkeypatch.setenv("SPK_RESIDENT", env)
        spk.spk_execute_solve(pl, to_dev(inputs.rhs(A.n_rows, 1)), x)
        modes.append(spk.spk_plan_get_info(pl)["exec_mode"])
    spk.spk_free(pl)
    assert modes == [spk.EXEC_RESIDENT, spk.EXEC_HOST_LOOP]


def test_split_products(spk, ctx, monkeypatch):
    A = ragged(3001, 50001, 14, 4)
    far = ragged(3001, 50001, 14, 4)
    far.row_ptr[1:] += 70_000        # row 0 holds 70,000 entries more, so row 1 starts past the packed offsets
    far = inputs.CSR(3001, 50001, far.row_ptr, np.resize(far.col, far.row_ptr[-1]), np.resize(far.val, far.row_ptr[-1]))

    def codes(M):
        pl = spk.spk_plan_spmv(ctx, M)
        out = spk.spk_plan_get_info(pl)["col_codes"]
        spk.spk_free(pl)
        return out

    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream,split=1")
    assert codes(dev_csr(spk, A)) == 0               # below 2^22 entries
    monkeypatch.setenv("SPK_SPLIT", "1")
    assert codes(dev_csr(spk, A)) == 8 and codes(dev_csr(spk, far)) == 0
    M = dev_csr(spk, A)
    odd = torch.empty(A.nnz + 1, dtype=torch.float64, device=DEV)
    odd[1:] = M.tensors[2]
    assert codes(spk.CsrMatrix(M.tensors[0], M.tensors[1], odd[1:], A.n_rows, A.n_cols)) == 0   # unaligned values
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream")
    assert codes(dev_csr(spk, A)) == 0
