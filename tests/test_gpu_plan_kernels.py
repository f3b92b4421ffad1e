"""Plan-time kernels that give a structure up while their workgroups start:
column codes whose missing offset most workgroups find, and row patterns with
rows too many to name, are dropped as a whole, and products come from the plain
indices or the codes, bit for bit (rows sum in the same order)."""
import numpy as np
import pytest
import torch

import inputs
from tests.gpu_util import DEV, dev_csr, to_dev
from tests.test_gpu_codes import banded

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


def product(spk, ctx, monkeypatch, A, codes, kernel):
    monkeypatch.setenv("SPK_COL_CODES", codes)
    monkeypatch.setenv("SPK_SPMV_KERNEL", kernel)
    pl = spk.spk_plan_spmv(ctx, dev_csr(spk, A))
    info = spk.spk_plan_get_info(pl)
    y = torch.full((A.n_rows,), float("nan"), dtype=torch.float64, device=DEV)
    spk.spk_execute_spmv(pl, to_dev(inputs.vec(A.n_cols, 1, 5)), y)
    spk.spk_free(pl)
    return y, info["col_codes"]


def two_bands(n, seed):
    """Every eighth tile of 256 rows (the ones sampled for offsets) has the offsets -1, 0, 1, the others 300 more
    between them, so that nearly every workgroup of the encoder meets a missing one."""
    rng = np.random.default_rng(seed)
    rows = np.arange(n)
    sampled = (rows // 256) % 8 == 0
    off = np.where(sampled, 0, 2 + rows % 300)
    cols = np.stack([np.clip(rows - 1, 0, n - 1), rows, np.clip(rows + 1, 0, n - 1), np.clip(rows + off, 0, n - 1)], 1)
    rp = np.arange(n + 1, dtype=np.int64) * 4
    return inputs.CSR(n, n, rp, cols.ravel().astype(np.int32), rng.uniform(-1, 1, 4 * n))


def test_codes_given_up(spk, ctx, monkeypatch):
    A = two_bands(600_001, 3)
    plain, c0 = product(spk, ctx, monkeypatch, A, "0", "stream")
    same, c1 = product(spk, ctx, monkeypatch, A, "1", "stream")
    assert c0 == 0 and c1 == 0 and torch.equal(same, plain)


@pytest.mark.parametrize("length", [8, 9, 64])
def test_long_patterns_checked(spk, ctx, monkeypatch, length):
    """Rows whose patterns are found by a hash and checked entry by entry, over many workgroups."""
    A = banded(300_001, list(range(-(length // 2), length - length // 2)), 5)
    plain, _ = product(spk, ctx, monkeypatch, A, "1", "stream,pats=0")
    same, c1 = product(spk, ctx, monkeypatch, A, "1", "stream,pats=1")
    # 64 offsets: the rows at the ends make 3,104 offsets in all, past the table's 1,024
    assert c1 == (3 if length == 64 else 7) and torch.equal(same, plain)


def test_many_patterns_named_by_many_waves(spk, ctx, monkeypatch):
    """256 distinct rows of 0 to 8 entries, every one of them in every workgroup: the waves share what they have
    seen of the table while it fills."""
    n, kinds = 300_001, 256
    kind = (np.arange(n) * 97) % kinds
    bits = (kind[:, None] >> np.arange(8)[None, :]) & 1
    cols = (np.arange(n)[:, None] + np.arange(8)[None, :])[bits == 1].astype(np.int32)
    rp = np.zeros(n + 1, np.int64)
    np.cumsum(bits.sum(1), out=rp[1:])
    A = inputs.CSR(n, n + 8, rp, cols, np.random.default_rng(5).uniform(-1, 1, cols.size))
    plain, _ = product(spk, ctx, monkeypatch, A, "1", "stream,pats=0")
    for _ in range(3):
        same, c1 = product(spk, ctx, monkeypatch, A, "1", "stream,pats=1")
        assert c1 == 7 and torch.equal(same, plain)
