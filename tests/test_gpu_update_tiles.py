"""GPU parity: the dense factor's update tiles at their edges -- leading
dimensions and addresses of every alignment, partial tiles in both directions,
both tile heights, right-hand sides of every chunk width."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, fwd_err, host

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _default_tuning():
    yield
    ebv.set_dense_tuning()


def _factor_solve(A, B, dtype, pad, off):
    """ebv_lu_factor_solve on a copy of A with lda = n + pad, `off` elements
    past an aligned address; the gap must come back untouched."""
    n, nrhs = B.shape
    buf = torch.full((off + n * (n + pad),), 3.0, dtype=dtype, device="cuda")
    view = buf[off:].view(n, n + pad)
    view[:, :n] = torch.from_numpy(A).to("cuda", dtype)
    X = torch.from_numpy(B).to("cuda", dtype)
    info = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    dt = ebv.F64 if dtype == torch.float64 else ebv.F32
    w, wb = ebv._ws_args(ebv.workspace(ebv.OP_FACTOR_SOLVE, dt, n, nrhs))
    rc = ebv.lib().ebv_lu_factor_solve(ebv.handle(), dt, n, nrhs, ebv._p(view), n + pad, ebv._p(X), nrhs,
                                       ebv._p(info), w, wb, ebv._stream())
    torch.cuda.synchronize()
    assert rc == 0 and int(info.item()) == 0
    assert bool((buf[:off] == 3.0).all()) and bool((view[:, n:] == 3.0).all())
    return host(view[:, :n]).astype(np.float64), host(X).astype(np.float64)


@pytest.mark.parametrize("tuning", [(0, True, 3, 0), (4096, True, 2, 0), (0, False, 1, 0), (4096, False, 1, 0)])
@pytest.mark.parametrize("n,nrhs,pad,off", [(129, 1, 0, 1), (191, 63, 1, 0), (192, 64, 2, 2), (321, 65, 3, 1),
                                            (449, 5, 63, 3)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_update_tiles(n, nrhs, pad, off, tuning, dtype):
    case(f"update tiles n={n} nrhs={nrhs} pad={pad} off={off} tuning={tuning} {dtype}")
    A, B = inputs.dense(n, 0.5, n), inputs.rhs(n, nrhs, n + 1)
    if dtype == torch.float32:
        A, B = (x.astype(np.float32).astype(np.float64) for x in (A, B))
    X_ref, LU_ref, _ = oracle.solve(A, B)
    ebv.set_dense_tuning(*tuning)
    LU, X = _factor_solve(A, B, dtype, pad, off)
    # entries of the factors are O(1) and kappa <= 3: n eps bounds both, with
    # a margin of 4
    tol = 1e-12 if dtype == torch.float64 else 4 * n * 6e-8
    assert np.abs(LU - LU_ref).max() <= tol
    assert fwd_err(X, X_ref) <= tol
