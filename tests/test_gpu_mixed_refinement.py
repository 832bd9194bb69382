"""GPU parity: the mixed-precision refinement's passes at their edges -- fewer
rows than a workgroup takes, every grouping of the right-hand sides, values
that are not numbers."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, fwd_err, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nrhs", [(1, 1), (3, 2), (7, 9), (9, 5), (255, 8), (257, 1), (513, 17), (1025, 4)])
def test_mixed_refinement(n, nrhs):
    case(f"mixed refinement n={n} nrhs={nrhs}")
    A, B = inputs.dense(n, 0.9, n), inputs.rhs(n, nrhs, n + 1)
    X_ref, _, _ = oracle.solve(A, B)
    X, iters, ferr, info = ebv.solve_mixed(dev(A), dev(B))
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    it = host(iters)
    assert it.min() >= 0 and it.max() <= 4
    assert host(ferr).max() <= 1e-12 and fwd_err(host(X), X_ref) <= 1e-12


def test_mixed_not_a_number():
    """A right-hand side with a NaN never converges; the others do."""
    n, nrhs = 200, 5
    case("mixed refinement with a NaN")
    A, B = inputs.dense(n, 0.5, 3), inputs.rhs(n, nrhs, 4)
    X_ref, _, _ = oracle.solve(A, B)
    B[17, 2] = np.nan
    X, iters, ferr, info = ebv.solve_mixed(dev(A), dev(B), max_iter=3)
    torch.cuda.synchronize()
    good = [0, 1, 3, 4]
    assert int(info.item()) == 0 and host(iters)[2] == -1 and host(iters)[good].min() >= 0
    assert not host(ferr)[2] <= 1e-12
    assert fwd_err(host(X)[:, good], X_ref[:, good]) <= 1e-12


def test_mixed_no_corrections():
    """max_iter = 0: the float solution and one test of it."""
    n = 130
    case("mixed refinement without corrections")
    A, B = inputs.dense(n, 0.5, 5), inputs.rhs(n, 3, 6)
    X_ref, _, _ = oracle.solve(A, B)
    X, iters, ferr, _ = ebv.solve_mixed(dev(A), dev(B), max_iter=0)
    torch.cuda.synchronize()
    err = fwd_err(host(X), X_ref)
    assert host(iters).max() == -1 and 1e-12 < host(ferr).max() and err <= host(ferr).max() <= 1e-4
