"""GPU parity: the factor in block steps, which large FP32 systems and calls
with more right-hand sides than the one launch has flags for take by default,
with the launches counted so that a test cannot pass on the other path.

Rows sum to 1.5 with the diagonal 1: no growth, kappa <= 3; errors are below
n eps for the factors and 4 n eps for the solutions (FP64 keeps the 1e-12 of
the other dense tests)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, host

pytestmark = pytest.mark.gpu

DTYPES = [torch.float64, torch.float32]


def _run(A, X0, dtype):
    """Factor + solve; returns L\\U, the solution, info and the launches of the elimination."""
    LU = dev(A, dtype)
    B = (LU.double() @ X0.double()).to(dtype)
    ebv.profile_update_enable(256)
    try:
        info = ebv.lu_factor_solve_(LU, B)
        torch.cuda.synchronize()
        launches = ebv.profile_update_read()[1]
    finally:
        ebv.profile_update_enable(0)
    return LU, B, int(info.item()), launches


def _check(A, X0, dtype, LU, X, info):
    n, eps = len(A), torch.finfo(dtype).eps
    LU_ref, _ = oracle.lu_factor(A.astype(np.float32).astype(np.float64) if dtype == torch.float32 else A)
    tol = 1e-12 if dtype == torch.float64 else n * eps
    assert info == 0
    assert np.abs(host(LU).astype(np.float64) - LU_ref).max() <= tol
    assert float((X.double() - X0.double()).abs().max()) <= 4 * max(n, 64) * eps * float(X0.abs().max())


@pytest.mark.parametrize("nrhs,steps", [(2304, False), (2305, True), (2400, True)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_block_steps_by_default(dtype, nrhs, steps):
    """24 block rows have 64 control words: four, a strip flag per block row and
    one per 64 right-hand sides.  The trailing block passes the size at which the
    steps go over from column classes to full updates (1024)."""
    n = 1500
    case(f"block steps by default nrhs={nrhs} {dtype}")
    A = inputs.dense(n, 0.5, 17)
    X0 = torch.rand((n, nrhs), dtype=dtype, device="cuda") - 0.5
    ebv.set_dense_tuning()
    LU, X, info, launches = _run(A, X0, dtype)
    assert launches == (23 if steps else 1)
    _check(A, X0, dtype, LU, X, info)


# (small_update_below, lookahead, defer_group, defer_above): every column in
# every launch; classes to the end, FP32 with 128-row and with 64-row tiles
@pytest.mark.parametrize("cfg", [(0, True, 1, 0), (0, True, 2, 0), (2048, True, 4, 0)])
@pytest.mark.parametrize("n,nrhs", [(64, 1), (65, 3), (300, 5), (700, 70)])
@pytest.mark.parametrize("dtype", DTYPES)
def test_block_steps_forced(dtype, n, nrhs, cfg):
    case(f"block steps forced n={n} nrhs={nrhs} {cfg} {dtype}")
    A = inputs.dense(n, 0.5, 18 + n)
    X0 = torch.rand((n, nrhs), dtype=dtype, device="cuda") - 0.5
    ebv.set_dense_tuning(*cfg)
    try:
        LU, X, info, launches = _run(A, X0, dtype)
    finally:
        ebv.set_dense_tuning()
    assert launches == (n + 63) // 64 - 1
    _check(A, X0, dtype, LU, X, info)


@pytest.mark.parametrize("n,nrhs", [(65, 3), (129, 8), (300, 70)])
def test_schemes_agree(n, nrhs):
    """Phases, look-ahead steps and the one launch give the same factor up to
    rounding order."""
    case(f"dense schemes agree n={n} nrhs={nrhs}")
    A = inputs.dense(n, 0.5, 19 + n)
    X0 = torch.rand((n, nrhs), dtype=torch.float64, device="cuda") - 0.5
    got = []
    for cfg in ((0, False, 1, 1024), (0, True, 3, 0), (0, True, 3, 1024)):
        ebv.set_dense_tuning(*cfg)
        try:
            got.append(_run(A, X0, torch.float64))
        finally:
            ebv.set_dense_tuning()
    assert [g[3] for g in got] == [(n + 63) // 64 - 1, (n + 63) // 64 - 1, 1]
    for LU, X, info, _ in got:
        assert info == 0
        assert float((LU - got[0][0]).abs().max()) <= 1e-13
        assert float((X - X0).abs().max()) <= 1e-12
