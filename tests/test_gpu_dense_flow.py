"""GPU parity of the one-launch factor of small systems at its edges: one to 32
block rows and one more (which takes block steps), partial last blocks, leading
dimensions and offsets that leave tiles sharing cache lines, no, one and
several block columns of right-hand sides, and zero pivots.

Entries of the factors are O(1) and kappa <= 3: n eps bounds the errors, with
a margin of 4 in FP32; FP64 keeps the 1e-12 of the other dense tests."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, fwd_err, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nrhs,pad,off", [(1, 1, 0, 0), (63, 2, 1, 1), (64, 64, 0, 0), (65, 65, 3, 0), (128, 1, 2, 1),
                                            (130, 130, 5, 3), (255, 17, 1, 0), (449, 200, 7, 1), (1023, 3, 0, 1),
                                            (1531, 1, 2, 0), (2048, 16, 0, 0), (2049, 1, 0, 0)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_dense_flow(n, nrhs, pad, off, dtype):
    case(f"dense flow n={n} nrhs={nrhs} pad={pad} off={off} {dtype}")
    A, B = inputs.dense(n, 0.5, n), inputs.rhs(n, nrhs, n + 1)
    if dtype == torch.float32:
        A, B = (x.astype(np.float32).astype(np.float64) for x in (A, B))
    X_ref, LU_ref, _ = oracle.solve(A, B)
    tol = 1e-12 if dtype == torch.float64 else 4 * max(n, 8) * 6e-8
    dt = ebv.F64 if dtype == torch.float64 else ebv.F32
    for rep in range(3):
        buf = torch.full((off + n * (n + pad),), 3.0, dtype=dtype, device="cuda")
        view = buf[off:].view(n, n + pad)
        view[:, :n] = torch.from_numpy(A).to("cuda", dtype)
        X = torch.from_numpy(B).to("cuda", dtype)
        info = torch.full((1,), 9, dtype=torch.int32, device="cuda")
        if rep < 2:
            w, wb = ebv._ws_args(ebv.workspace(ebv.OP_FACTOR_SOLVE, dt, n, nrhs))
            rc = ebv.lib().ebv_lu_factor_solve(ebv.handle(), dt, n, nrhs, ebv._p(view), n + pad, ebv._p(X), nrhs,
                                               ebv._p(info), w, wb, ebv._stream())
        else:  # without right-hand sides
            w, wb = ebv._ws_args(ebv.workspace(ebv.OP_FACTOR, dt, n, 0))
            rc = ebv.lib().ebv_lu_factor(ebv.handle(), dt, n, ebv._p(view), n + pad, 1, 0, ebv._p(info), w, wb,
                                         ebv._stream())
        torch.cuda.synchronize()
        assert rc == 0 and int(info.item()) == 0
        assert bool((buf[:off] == 3.0).all()) and bool((view[:, n:] == 3.0).all())
        assert np.abs(host(view[:, :n]).astype(np.float64) - LU_ref).max() <= tol
        if rep < 2:
            assert fwd_err(host(X).astype(np.float64), X_ref) <= tol


@pytest.mark.parametrize("zeros", [(0,), (200, 70), (333,)])
def test_dense_flow_zero_pivot(zeros):
    """A diagonal matrix with zeros: the smallest zero pivot is reported."""
    case(f"dense flow zero pivots {zeros}")
    d = torch.ones(350, dtype=torch.float64, device="cuda")
    d[list(zeros)] = 0.0
    A = torch.diag(d).contiguous()
    assert int(ebv.lu_factor_(A).item()) == min(zeros) + 1
