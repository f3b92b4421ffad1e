"""CG loops whose vectors outgrow the last-level cache (60 MiB and more each):
x goes past the cache and the passes run backwards.  Solves on both sides of
the line, with odd remainders and an unaligned solution vector (which takes
the loop of single values), against the solution the right-hand side was made
from."""
import pytest
import torch

from tests.gpu_util import DEV

pytestmark = pytest.mark.gpu

EDGE64, EDGE32 = (60 << 20) // 8, (60 << 20) // 4


@pytest.fixture(scope="module")
def spk():
    from paper_2510_08230_amd import spk as m
    return m


@pytest.fixture(scope="module")
def ctx(spk):
    c = spk.spk_init(0, torch.cuda.current_stream().cuda_stream)
    yield c
    spk.spk_finalize(c)


def tridiagonal(spk, n, diag):
    """diag on the diagonal (a vector), -1 beside it."""
    i = torch.arange(n, dtype=torch.int64, device=DEV)
    rp = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    rp[1:] = torch.cumsum(3 - (i == 0).long() - (i == n - 1).long(), 0)
    ci = torch.stack((i - 1, i, i + 1), 1).reshape(-1)[1:-1].to(torch.int32)
    va = torch.stack((torch.full_like(diag, -1.0), diag, torch.full_like(diag, -1.0)), 1).reshape(-1)[1:-1].contiguous()
    return spk.CsrMatrix(rp, ci.contiguous(), va, n, n)


@pytest.mark.parametrize("n,precision,jacobi,shift", [
    (EDGE64 - 1, "fp64", False, 0), (EDGE64, "fp64", False, 0), (EDGE64 + 1, "fp64", False, 0),
    (EDGE64 + 1, "fp64", False, 1), (EDGE64 - 1, "fp64", True, 0), (EDGE64 + 1, "fp64", True, 0),
    (EDGE64 + 1, "fp64", True, 1), (EDGE32 - 1, "mixed_fp32", False, 0), (EDGE32 + 3, "mixed_fp32", False, 0)])
def test_solves_at_the_line(spk, ctx, n, precision, jacobi, shift):
    gen = torch.Generator(device=DEV).manual_seed(n)
    diag = 4.0 + torch.rand(n, dtype=torch.float64, device=DEV, generator=gen)
    want = torch.rand(n, dtype=torch.float64, device=DEV, generator=gen) - 0.5
    b = diag * want
    b[1:] -= want[:-1]
    b[:-1] -= want[1:]
    cfg = spk.spk_solver_cfg_default()
    cfg.solver = spk.SOLVER_CG
    cfg.precond = spk.PRECOND_JACOBI if jacobi else spk.PRECOND_NONE
    cfg.precision = {"fp64": spk.PREC_FP64, "mixed_fp32": spk.PREC_MIXED_FP32}[precision]
    cfg.reduction_factor = 1e-10
    pl = spk.spk_plan_solve(ctx, tridiagonal(spk, n, diag), cfg)
    for _ in range(2):
        x = torch.zeros(n + shift, dtype=torch.float64, device=DEV)[shift:]
        log = spk.spk_execute_solve(pl, b, x)
        assert log.stop_reason == spk.STOP_CONVERGED
        # eigenvalues in [2, 7]: ||x - want|| <= tau ||b|| / 2 <= 3.5 tau ||want||
        assert float((x - want).norm() / want.norm()) <= 3.5e-10
    spk.spk_free(pl)
