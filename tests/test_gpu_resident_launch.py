"""How a plan's resident launch (one launch per small CG solve) is told from
the loop that takes its place: every solve of a plan whose launches are refused, or
whose waits time out, equals the loop's, whatever its number, caps and chunk
length.  (A time-out is a mark set from the host: the launch itself runs as
usual and stores x, which has to be put back.)"""
import pytest
import torch

import inputs
from tests.gpu_util import DEV, dev_csr, to_dev
from tests.test_gpu_resident import band

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
    for name in ("SPK_CG_FUSED", "SPK_SPMV_KERNEL", "SPK_RESIDENT", "SPK_LONG_ROWS"):
        monkeypatch.delenv(name, raising=False)


def config(spk, precision, max_iters=1000, chunk=0):
    cfg = spk.spk_solver_cfg_default()
    cfg.precision = spk.PREC_FP64 if precision == "fp64" else spk.PREC_MIXED_FP32
    cfg.reduction_factor = 1e-12
    cfg.max_iters = max_iters
    cfg.chunk_iters = chunk
    return cfg


def plan(spk, ctx, monkeypatch, M, cfg, resident):
    monkeypatch.setenv("SPK_RESIDENT", resident)
    return spk.spk_plan_solve(ctx, M, cfg)


def solve(spk, pl, b, x0):
    x = x0.clone()
    log = spk.spk_execute_solve(pl, b, x)
    return x, log


def same(got, want):
    return (torch.equal(got[0], want[0]) and got[1].iterations == want[1].iterations
            and got[1].stop_reason == want[1].stop_reason and got[1].implicit_resnorm == want[1].implicit_resnorm
            and got[1].rhs_norm == want[1].rhs_norm)


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
@pytest.mark.parametrize("max_iters,chunk", [(1000, 0), (1000, 1), (1, 0), (1, 1), (5, 2)])
def test_every_refused_launch_is_followed_by_the_loop(spk, ctx, monkeypatch, precision, max_iters, chunk):
    A = inputs.stencil7(8, 1)
    M = dev_csr(spk, A)
    cfg = config(spk, precision, max_iters, chunk)
    loop = plan(spk, ctx, monkeypatch, M, cfg, "0")
    refused = plan(spk, ctx, monkeypatch, M, cfg, "refuse")
    x0 = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    for k in range(100):
        b = to_dev(inputs.vec(A.n_rows, 1, k))
        ok = same(solve(spk, refused, b, x0), solve(spk, loop, b, x0))
        if not ok:
            break
    spk.spk_free(loop)
    spk.spk_free(refused)
    assert ok, k


def test_profiled_solves_do_not_pass_for_a_launch(spk, ctx, monkeypatch):
    """A profiled solve runs the loop too: its counters are not taken for the next launch's number."""
    A = inputs.stencil7(8, 1)
    M = dev_csr(spk, A)
    cfg = config(spk, "fp64", 1, 1)
    loop = plan(spk, ctx, monkeypatch, M, cfg, "0")
    pl = plan(spk, ctx, monkeypatch, M, cfg, "refuse")
    x0 = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    good = []
    for k in range(8):
        b = to_dev(inputs.vec(A.n_rows, 2, k))
        spk.spk_plan_set_profiling(pl, 1)
        first = solve(spk, pl, b, x0)
        spk.spk_plan_set_profiling(pl, 0)
        want = solve(spk, loop, b, x0)
        good.append(same(first, want) and same(solve(spk, pl, -b, x0), solve(spk, loop, -b, x0)))
    spk.spk_free(loop)
    spk.spk_free(pl)
    assert all(good), good


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
@pytest.mark.parametrize("half", [3, 4, 5, 15, 16])
def test_without_the_long_row_pass(spk, ctx, monkeypatch, precision, half):
    """SPK_LONG_ROWS=0 leaves long rows to one lane; it does not change what a resident solve knows of its rows
    (their entries past the registers' eight are kept in LDS), so solves are the same bit for bit."""
    A = band(300, half, 4)
    M = dev_csr(spk, A)
    b = to_dev(inputs.rhs(A.n_rows, 4))
    x0 = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    out = []
    for long_rows in ("1", "0"):
        monkeypatch.setenv("SPK_LONG_ROWS", long_rows)
        pl = plan(spk, ctx, monkeypatch, M, config(spk, precision), "1")
        out.append(solve(spk, pl, b, x0))
        spk.spk_free(pl)
    assert out[0][1].stop_reason == spk.STOP_CONVERGED and same(out[1], out[0])


@pytest.mark.parametrize("precision", ["fp64", "mixed_fp32"])
@pytest.mark.parametrize("kind,size", [("stencil7", 8), ("band", 4097)])
def test_after_a_timeout_the_plan_stays_with_the_loop(spk, ctx, monkeypatch, precision, kind, size):
    A = inputs.stencil7(size, 1) if kind == "stencil7" else band(size, 4, 1)
    M = dev_csr(spk, A)
    loop = plan(spk, ctx, monkeypatch, M, config(spk, precision), "0")
    pl = plan(spk, ctx, monkeypatch, M, config(spk, precision), "1")
    x0 = to_dev(inputs.vec(A.n_rows, 1, 9))
    good = []
    for k, mode in enumerate(("refuse", "timeout", "1", "refuse", "1")):
        b = to_dev(inputs.vec(A.n_rows, 3, k))
        monkeypatch.setenv("SPK_RESIDENT", mode)
        got = solve(spk, pl, b, x0)
        want = solve(spk, loop, b, x0)
        good.append(got[1].stop_reason == spk.STOP_CONVERGED and same(got, want))
    spk.spk_free(loop)
    spk.spk_free(pl)
    assert all(good), good


def test_noalloc_solve_after_a_timeout(spk, ctx, monkeypatch):
    A = band(4097, 4, 1)
    M = dev_csr(spk, A)
    b, x0 = to_dev(inputs.rhs(A.n_rows, 3)), to_dev(inputs.vec(A.n_rows, 1, 9))
    out = []
    for mode in ("0", "timeout", "refuse"):
        monkeypatch.setenv("SPK_RESIDENT", mode)
        x = x0.clone()
        out.append((x, spk.spk_solve_noalloc(ctx, M, b, x, config(spk, "fp64"))))
    assert same(out[1], out[0]) and same(out[2], out[0])
