"""Rows of more than 256 entries are summed in pieces of at most 1,024 by a
launch of their own ahead of the row tiles (CSR and COO), or, where a call
has no memory for the list of pieces, in the tile itself in the same order.

Dyadic values and small-integer x make every partial sum exact in FP32 and
FP64 (at most 5,000 terms below 2^4 with 1 fractional bit), so products at the
pieces' edges equal the oracle's bit for bit; the allocation-free solve, which
has no list, equals a planned solve bit for bit."""
import numpy as np
import pytest
import torch

import inputs
import oracle
from tests.gpu_util import DEV, TORCH_IDX, dev_csr, to_dev
from tests.test_gpu_long_rows import dyadic_hubs

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


@pytest.fixture(scope="module")
def hubs():
    # distinct columns are drawn, so the lengths land near the figure: pad to it exactly
    A = dyadic_hubs(6000, 5, {})
    lens = {0: 256, 1: 257, 255: 1023, 256: 1024, 300: 1025, 2500: 2048, 2501: 2049, 5999: 5000}
    rp, cols, vals = [0], [], []
    for i in range(A.n_rows):
        m = lens.get(i)
        if m is None:
            a, b = A.row_ptr[i], A.row_ptr[i + 1]
            cols.append(A.col[a:b])
            vals.append(A.val[a:b])
        else:
            cols.append(np.arange(m, dtype=np.int32))
            vals.append(np.resize(np.array([0.5, -1.0, 1.0, -0.5, 1.0]), m))
        rp.append(rp[-1] + len(cols[-1]))
    return inputs.CSR(A.n_rows, A.n_cols, np.array(rp, np.int64), np.concatenate(cols).astype(np.int32),
                      np.concatenate(vals))


@pytest.mark.parametrize("fmt", ["csr", "coo"])
@pytest.mark.parametrize("val", [torch.float64, torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("idx", ["i32", "i64"])
def test_piece_edges_bit_exact(spk, ctx, monkeypatch, hubs, fmt, val, idx):
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream")
    x = np.array([float((inputs.hash64(5, 13, j) % 17) - 8) for j in range(hubs.n_cols)])
    vt = torch.float64 if val == torch.float64 else torch.float32
    if fmt == "csr":
        pl = spk.spk_plan_spmv(ctx, dev_csr(spk, hubs, idx, idx, val))
    else:
        rows = np.repeat(np.arange(hubs.n_rows), np.diff(hubs.row_ptr))
        M = spk.CooMatrix(torch.from_numpy(rows).to(TORCH_IDX[idx]).to(DEV),
                          torch.from_numpy(hubs.col).to(TORCH_IDX[idx]).to(DEV), to_dev(hubs.val, val), hubs.n_rows,
                          hubs.n_cols)
        pl = spk.spk_plan_spmv_coo(ctx, M)
    y = torch.full((hubs.n_rows,), float("nan"), dtype=vt, device=DEV)
    for _ in range(2):
        spk.spk_execute_spmv(pl, to_dev(x, vt), y)
        assert np.array_equal(y.double().cpu().numpy(), oracle.spmv(hubs, x))
    spk.spk_free(pl)


@pytest.mark.parametrize("n", [30000, 150000])
def test_in_tile_sums_equal_pieces(spk, ctx, monkeypatch, n):
    monkeypatch.setenv("SPK_SPMV_KERNEL", "stream")
    monkeypatch.delenv("SPK_CG_FUSED", raising=False)
    A = inputs.powerlaw(n, 4)
    M = dev_csr(spk, A, "i32", "i32")
    b = to_dev(inputs.rhs(n, 4))
    cfg = spk.spk_solver_cfg_default()
    cfg.max_iters = 20
    cfg.reduction_factor = 0.0
    pl = spk.spk_plan_solve(ctx, M, cfg)
    xp = torch.zeros(n, dtype=torch.float64, device=DEV)
    spk.spk_execute_solve(pl, b, xp)
    spk.spk_free(pl)
    xn = torch.zeros(n, dtype=torch.float64, device=DEV)
    spk.spk_solve_noalloc(ctx, M, b, xn, cfg)
    assert np.array_equal(xn.cpu().numpy().view(np.uint64), xp.cpu().numpy().view(np.uint64))
