"""Matrices of one size and type share the tuner's result only where they have
the same structures (row patterns, split gathers): a plan without one does not
decide for a later plan that has it, nor the other way round."""
import numpy as np
import pytest
import torch

import inputs
from tests.gpu_util import dev_csr

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def spk():
    from paper_2510_08230_amd import spk as m
    return m


@pytest.fixture
def ctx(spk):
    c = spk.spk_init(0, torch.cuda.current_stream().cuda_stream)   # an empty cache
    yield c
    spk.spk_finalize(c)


@pytest.fixture(autouse=True)
def plain_env(monkeypatch):
    for name in ("SPK_SPMV_KERNEL", "SPK_COL_CODES", "SPK_ROW_PATTERNS", "SPK_SPLIT", "SPK_LONG_ROWS"):
        monkeypatch.delenv(name, raising=False)


def info(spk, ctx, A):
    pl = spk.spk_plan_spmv(ctx, dev_csr(spk, A, "i32", "i32", torch.float32))
    out = spk.spk_plan_get_info(pl)
    spk.spk_free(pl)
    return out


@pytest.fixture(scope="module")
def grid():
    """A 7-point stencil, and the same rows with their entries in random orders (too many distinct rows)."""
    A = inputs.stencil7(128, 1)
    key = np.repeat(np.arange(A.n_rows, dtype=np.float64), np.diff(A.row_ptr))
    order = np.argsort(key + np.random.default_rng(2).random(A.nnz), kind="stable")
    return A, inputs.CSR(A.n_rows, A.n_cols, A.row_ptr, A.col[order], A.val[order])


@pytest.mark.parametrize("first", ["patterns", "none"])
def test_patterns(spk, ctx, grid, first):
    A, B = grid
    if first == "patterns":
        a, b = info(spk, ctx, A), info(spk, ctx, B)
    else:
        b, a = info(spk, ctx, B), info(spk, ctx, A)
    # the pattern kernel is a fifth faster at this size; codes with and without packed rows tie
    assert a["col_codes"] == 7 and b["col_codes"] in (1, 3)
    assert a["spmv_ms"] != b["spmv_ms"]


def seven_per_row(n, at, length, seed):
    """Seven entries per row at random columns, row `at` holding `length`."""
    lens = np.full(n, 7)
    lens[at] = length
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    nnz = int(rp[-1])
    rng = np.random.default_rng(seed)
    return inputs.CSR(n, n, rp, rng.integers(0, n, nnz, dtype=np.int32), np.ones(nnz))


def test_split(spk, ctx):
    # row 1 starts 70,000 entries into its tile: no packed row pointers, so no split; as the tile's last row they fit
    without = info(spk, ctx, seven_per_row(3_000_000, 0, 70_000, 1))
    split = info(spk, ctx, seven_per_row(3_000_000, 255, 70_000, 1))
    assert split["spmv_ms"] < 0.8 * without["spmv_ms"]   # 102 against 228 us without the long row
    assert info(spk, ctx, seven_per_row(3_000_000, 0, 70_000, 1))["spmv_ms"] == without["spmv_ms"]
