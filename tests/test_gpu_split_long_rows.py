"""Rows of more than 256 entries in tiles that fit the LDS stage, with the
gathers ahead in column order: their sums are those of the plain row tiles
(the row's pieces in order), so products agree bit for bit."""
import numpy as np
import pytest
import torch

import inputs
from tests.gpu_util import DEV, dev_csr, to_dev

pytestmark = pytest.mark.gpu

N, COLS = 3001, 50001
# a row per tile of 256 rows; with 0 to 2 entries in the others its tile stays below 2,048 entries; the last one
# is its tile's only row past the others' and shares the ragged tile
LONG = {0: 257, 300: 300, 600: 500, 800: 1000, 1100: 1024, 1300: 1025, 1700: 1500, 2047: 256, 3000: 700}


@pytest.fixture(scope="module")
def spk():
    from paper_2510_08230_amd import spk as m
    return m


@pytest.fixture(scope="module")
def ctx(spk):
    c = spk.spk_init(0, torch.cuda.current_stream().cuda_stream)
    yield c
    spk.spk_finalize(c)


def matrix(seed):
    rng = np.random.default_rng(seed)
    lens = rng.integers(0, 3, N)
    for i, m in LONG.items():
        lens[i] = m
    rp = np.zeros(N + 1, np.int64)
    np.cumsum(lens, out=rp[1:])
    tiles = np.add.reduceat(lens, np.arange(0, N, 256))
    assert tiles.max() <= 2048
    nnz = int(rp[-1])
    return inputs.CSR(N, COLS, rp, rng.integers(0, COLS, nnz).astype(np.int32), rng.uniform(-1, 1, nnz))


def product(spk, ctx, monkeypatch, A, val, idx, kernel):
    monkeypatch.setenv("SPK_SPLIT", "1")
    monkeypatch.setenv("SPK_COL_CODES", "0")
    monkeypatch.setenv("SPK_SPMV_KERNEL", kernel)
    vt = torch.float64 if val == torch.float64 else torch.float32
    pl = spk.spk_plan_spmv(ctx, dev_csr(spk, A, idx, idx, val))
    y = torch.full((A.n_rows,), float("nan"), dtype=vt, device=DEV)
    for _ in range(2):
        spk.spk_execute_spmv(pl, to_dev(inputs.vec(A.n_cols, 1, 5), vt), y)
    spk.spk_free(pl)
    return y


@pytest.mark.parametrize("val", [torch.float64, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("idx", ["i32", "i64"])
def test_long_rows_in_staged_tiles(spk, ctx, monkeypatch, val, idx):
    A = matrix(3)
    plain = product(spk, ctx, monkeypatch, A, val, idx, "stream,remap=64")
    for opts in ("nt=1,remap=64", "nt=0,remap=0,bpc=16"):
        assert torch.equal(product(spk, ctx, monkeypatch, A, val, idx, "stream,split=1," + opts), plain)
