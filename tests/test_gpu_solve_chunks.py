"""GPU parity: right-hand sides in chunks of 16 solved side by side, with room
for all of them, for some and for one at a time."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, fwd_err, host

pytestmark = pytest.mark.gpu


def _ws(op, n, nrhs, room_for):
    """Workspace with room for `room_for` chunks."""
    return ebv.workspace(op, ebv.F64, n, 16 * room_for)


@pytest.mark.parametrize("n,nrhs,room", [(1, 17, 2), (64, 65, 4), (200, 33, 1), (200, 33, 2), (321, 64, 4),
                                         (321, 130, 3)])
def test_chunked_solves(n, nrhs, room):
    case(f"chunked solves n={n} nrhs={nrhs} room={room}")
    A, B = inputs.dense(n, 0.5, 10 + n), inputs.rhs(n, nrhs, 11 + n)
    X_ref, LU_ref, _ = oracle.solve(A, B)
    LU = dev(LU_ref)
    X, info = dev(B), torch.full((1,), 7, dtype=torch.int32, device="cuda")
    ebv.lu_solve_(LU, X, ws=_ws(ebv.OP_SOLVE, n, nrhs, room), info=info)
    G = inputs.rhs(n, nrhs, 12 + n)
    gB, _ = ebv.lu_solve_adjoint(LU, X, dev(G), want_abar=False, ws=_ws(ebv.OP_ADJOINT, n, nrhs, room))
    A2, X2 = dev(A), dev(B)
    info2 = ebv.lu_factor_solve_(A2, X2, ws=_ws(ebv.OP_FACTOR_SOLVE, n, nrhs, room))
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and int(info2.item()) == 0
    assert fwd_err(host(X), X_ref) <= 1e-13 and fwd_err(host(X2), X_ref) <= 1e-12
    assert fwd_err(host(gB), np.linalg.solve(A.T, G)) <= 1e-12


@pytest.mark.parametrize("room", [1, 3])
def test_chunked_mixed(room):
    n, nrhs = 200, 40
    case(f"chunked mixed solve room={room}")
    A, B = inputs.dense(n, 0.9, 21), inputs.rhs(n, nrhs, 22)
    X_ref, _, _ = oracle.solve(A, B)
    full = ebv.workspace(ebv.OP_MIXED, ebv.F64, n, nrhs)
    per = ebv.workspace(ebv.OP_SOLVE, ebv.F32, n, 32).numel() - ebv.workspace(ebv.OP_SOLVE, ebv.F32, n, 16).numel()
    ws = torch.empty(full.numel() - (3 - room) * per, dtype=torch.uint8, device="cuda")
    X, iters, _, info = ebv.solve_mixed(dev(A), dev(B), ws=ws)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and int(iters.min().item()) >= 0
    assert fwd_err(host(X), X_ref) <= 1e-12
