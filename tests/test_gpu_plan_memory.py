"""Structures that only make products faster (row patterns, the pieces of long
rows) give way to a solve's own vectors: a plan fits into the device memory in
which it fits without them.  Run in a child process whose hipMalloc refuses
what would pass a limit (alloc_limit.c)."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, os, sys
sys.path.insert(0, {root!r})
import numpy as np
import torch
import inputs, oracle
from paper_2510_08230_amd import spk
from tests.gpu_util import DEV, dev_csr, rel, to_dev
lim = ctypes.CDLL({shim!r})
for f in (lim.alloc_limit_used, lim.alloc_limit_peak):
    f.restype = ctypes.c_size_t
lim.alloc_limit_set.argtypes = [ctypes.c_size_t]
kind, solver = {kind!r}, {solver!r}
off = "SPK_ROW_PATTERNS" if kind == "patterns" else "SPK_LONG_ROWS"
os.environ["SPK_COL_CODES"] = "1" if kind == "patterns" else "0"   # (codes are tried where long rows are unknown)
os.environ["SPK_SPMV_KERNEL"] = "stream,pats=1"
A = inputs.stencil7(60, 1) if kind == "patterns" else inputs.powerlaw(200000, 7)
bh = inputs.rhs(A.n_rows, 1)
M, b, x = dev_csr(spk, A), to_dev(bh), torch.zeros(A.n_rows, dtype=torch.float64, device=DEV)
cfg = spk.spk_solver_cfg_default()
cfg.reduction_factor, cfg.max_iters = 1e-10, 5000
cfg.solver = spk.SOLVER_GMRES if solver == "gmres" else spk.SOLVER_CG
cfg.precision = spk.PREC_MIXED_FP32 if solver == "mixed" else spk.PREC_FP64

def run():
    ctx = spk.spk_init(0, torch.cuda.current_stream().cuda_stream)   # an empty pool
    try:
        pl = spk.spk_plan_solve(ctx, M, cfg)
        codes = spk.spk_plan_get_info(pl)["col_codes"]
        x.zero_()
        log = spk.spk_execute_solve(pl, b, x)
        spk.spk_free(pl)
    finally:
        spk.spk_finalize(ctx)
    assert log.stop_reason == spk.STOP_CONVERGED, log.stop_reason
    assert np.linalg.norm(oracle.residual(A, bh, x.cpu().numpy())) <= 1.01e-10 * np.linalg.norm(bh)
    return codes

def peak():
    lim.alloc_limit_reset_peak()
    codes = run()
    return lim.alloc_limit_peak(), codes

full, c1 = peak()
os.environ[off] = "0"
bare, c0 = peak()
del os.environ[off]
print(kind, solver, "bytes with", full, "without", bare, "codes", c1, c0, flush=True)
assert bare < full
if kind == "patterns":
    assert c1 == 7 and c0 == 3
lim.alloc_limit_set(bare)
c2 = run()   # no more than it takes without the structure
print("codes at the limit", c2, flush=True)
lim.alloc_limit_set(full)
assert run() == c1
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("shim") / "liballoc_limit.so")
    subprocess.check_call(["gcc", "-O2", "-shared", "-fPIC", os.path.join(ROOT, "tests", "alloc_limit.c"), "-o", out,
                           "-ldl"])
    return out


@pytest.mark.parametrize("kind", ["patterns", "pieces"])
@pytest.mark.parametrize("solver", ["cg", "gmres", "mixed"])
def test_structures_give_way(shim, kind, solver):
    env = dict(os.environ)
    env["LD_PRELOAD"] = " ".join(filter(None, [shim, env.get("LD_PRELOAD", "")]))
    r = subprocess.run([sys.executable, "-u", "-c", CHILD.format(root=ROOT, shim=shim, kind=kind, solver=solver)],
                       env=env, capture_output=True, text=True, timeout=100)
    print(r.stdout)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
