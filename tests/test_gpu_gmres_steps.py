"""The scalar work at the end of a GMRES step hands its column from the lanes
that form it to the one that rotates it: every step's residual estimate and the
iterates at the edges of the restart length (a term per lane, up to 33)
against the oracle.  Tolerances as for the other restart lengths: iterates of
a fixed number of steps within 1e-12, residual estimates within 1%."""
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


@pytest.mark.parametrize("m,K", [(1, 3), (2, 5), (31, 31), (32, 32), (32, 40)])
def test_steps(spk, ctx, m, K):
    A = inputs.stencil7_ns(20, 1, delta=0.2)
    b = inputs.rhs(A.n_rows, 1)
    cfg = spk.spk_solver_cfg_default()
    cfg.solver, cfg.krylov_dim, cfg.max_iters, cfg.reduction_factor, cfg.record_history = spk.SOLVER_GMRES, m, K, 0.0, 1
    pl = spk.spk_plan_solve(ctx, dev_csr(spk, A), cfg)
    x = torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
    log = spk.spk_execute_solve(pl, to_dev(b), x)
    hist = np.asarray(spk.spk_plan_history(pl))
    spk.spk_free(pl)
    xo, ro, ho = oracle.gmres(A, b, tau=0.0, max_iters=K, m=m, history=True)
    assert log.iterations == K and hist.size == ho.size == K + 1
    assert np.all(np.abs(hist - ho) <= 0.01 * ho)
    assert rel(x.cpu().numpy(), xo) <= 1e-12
