"""Row patterns (one byte per row naming its whole sequence of column offsets)
against column codes: rows sum in the same order on the same values, so
products agree bit for bit and solves give identical iterates.

Rows of 0, 7 (the longest whose key is exact), 8, 9 and 64 entries, 65 (no
patterns), 256 and 257 distinct rows, rare rows, ragged tails, tiles past the
LDS stage, unsorted and repeated columns."""
import numpy as np
import pytest
import torch

import inputs
from tests.gpu_util import DEV, dev_csr, to_dev
from tests.test_gpu_codes import MATS, banded

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
def codes_at_any_size(monkeypatch):
    monkeypatch.setenv("SPK_COL_CODES", "1")


def distinct_rows(n, kinds, seed):
    """Row i holds the offsets of the bits of i % kinds among -4..4, so there are `kinds` distinct interior rows;
    every row is interior (columns wrap no further than the matrix is wide)."""
    rng = np.random.default_rng(seed)
    rp, cols = [0], []
    for i in range(n):
        cols.extend(i + d for d in range(9) if (i % kinds) >> d & 1)
        rp.append(len(cols))
    return inputs.CSR(n, n + 9, np.array(rp, np.int64), np.array(cols, np.int32), rng.uniform(-1, 1, len(cols)))


def wide(n, k, seed):
    """Rows of k entries at the offsets 0..k-1 (one pattern)."""
    cols = (np.arange(n)[:, None] + np.arange(k)[None, :]).astype(np.int32)
    return inputs.CSR(n, n + k, np.arange(n + 1, dtype=np.int64) * k, cols.ravel(),
                      np.random.default_rng(seed).uniform(-1, 1, n * k))


def shuffled(A, seed):
    """The same rows with their entries in another order, the same in equal rows, and one column repeated."""
    cols, vals, rp = [], [], [0]
    for i in range(A.n_rows):
        a, b = A.row_ptr[i], A.row_ptr[i + 1]
        order = np.random.default_rng(seed + int(b - a)).permutation(b - a)
        c, v = A.col[a:b][order], A.val[a:b][order]
        cols.append(np.append(c, c[:1]))
        vals.append(np.append(v, 0.25 * v[:1]))
        rp.append(rp[-1] + len(cols[-1]))
    return inputs.CSR(A.n_rows, A.n_cols, np.array(rp, np.int64), np.concatenate(cols), np.concatenate(vals))


ALL = dict(MATS)
ALL.update({
    "band8": lambda: banded(2000, [-400, -20, -1, 0, 1, 2, 20, 400], 4),
    "wide64": lambda: wide(1200, 64, 5),
    "rows256": lambda: distinct_rows(4000, 256, 6),
    "shuffled": lambda: shuffled(inputs.stencil7(14, 2), 3),
    "one_row": lambda: banded(1, [0], 7),
})


def product(spk, ctx, monkeypatch, A, val, idx, kernel):
    monkeypatch.setenv("SPK_SPMV_KERNEL", kernel)
    vt = torch.float64 if val == torch.float64 else torch.float32
    pl = spk.spk_plan_spmv(ctx, dev_csr(spk, A, idx, idx, val))
    info = spk.spk_plan_get_info(pl)
    y = torch.full((A.n_rows,), float("nan"), dtype=vt, device=DEV)
    for _ in range(2):
        spk.spk_execute_spmv(pl, to_dev(inputs.vec(A.n_cols, 1, 5), vt), y)
    spk.spk_free(pl)
    return y, info["col_codes"]


@pytest.mark.parametrize("name", sorted(ALL))
@pytest.mark.parametrize("val", [torch.float64, torch.float32, torch.float16])
@pytest.mark.parametrize("idx", ["i32", "i64"])
def test_products_bit_equal(spk, ctx, monkeypatch, name, val, idx):
    A = ALL[name]()
    codes, c0 = product(spk, ctx, monkeypatch, A, val, idx, "stream,pats=0")
    assert c0 == 3
    for opts in ("", ",nt=1,remap=64", ",remap=0,bpc=16"):
        pats, c1 = product(spk, ctx, monkeypatch, A, val, idx, "stream,pats=1" + opts)
        assert c1 == 7 and torch.equal(pats, codes)


@pytest.mark.parametrize("name,make", [("rows257", lambda: distinct_rows(4000, 300, 6)),
                                       ("row65", lambda: wide(1200, 65, 5)),
                                       # 65 distinct rows, 3,104 offsets in all: past the table's 1,024
                                       ("band64", lambda: banded(1200, range(-32, 32), 5))])
def test_without_patterns(spk, ctx, monkeypatch, name, make):
    A = make()
    codes, c0 = product(spk, ctx, monkeypatch, A, torch.float64, "i32", "stream,pats=0")
    same, c1 = product(spk, ctx, monkeypatch, A, torch.float64, "i32", "stream,pats=1")
    assert c0 == 3 and c1 == 3 and torch.equal(same, codes)


@pytest.mark.parametrize("solver,precision,precond", [(0, 0, 0), (0, 1, 0), (0, 3, 0), (1, 0, 0), (2, 0, 0), (2, 1, 0),
                                                      (0, 0, 1), (2, 0, 1)])
def test_solves_identical(spk, ctx, monkeypatch, solver, precision, precond):
    A = inputs.stencil7(30, 3) if solver == 0 else inputs.stencil7_ns(30, 3)
    b = to_dev(inputs.vec(A.n_rows, 3, 2))
    cfg = spk.spk_solver_cfg_default()
    cfg.solver, cfg.precision, cfg.precond = solver, precision, precond
    cfg.reduction_factor = 1e-12
    cfg.inner_reduction = 1e-3
    out = []
    for kernel in ("stream,pats=0", "stream,pats=1"):
        monkeypatch.setenv("SPK_SPMV_KERNEL", kernel)
        pl = spk.spk_plan_solve(ctx, dev_csr(spk, A), cfg)
        x = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
        log = spk.spk_execute_solve(pl, b, x)
        spk.spk_free(pl)
        assert log.converged
        out.append((x, log.iterations))
    assert out[0][1] == out[1][1] and torch.equal(out[0][0], out[1][0])
