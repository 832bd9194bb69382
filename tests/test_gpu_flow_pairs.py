"""GPU parity of the one-launch factor in the order of pairs of steps (systems
beyond n = 7168), with an even and an odd number of block rows, a partial last
block and right-hand sides: the solution's residual and the factors' product
against the matrix, on the device in FP64.

Rows sum to at most 1.5 with the diagonal 1, so the elimination does not grow and
the product's error per element is below n eps; FP32 the same with its eps."""
from __future__ import annotations

import pytest
import torch

from paper_1907_05767_amd import ebv
from tests.gpu_util import case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nrhs,dtype", [(7232, 3, torch.float64), (7233, 70, torch.float32),
                                          (7300, 65, torch.float64)])
def test_flow_pairs(n, nrhs, dtype):
    case(f"flow pairs n={n} nrhs={nrhs} {dtype}")
    gen = torch.Generator(device="cuda").manual_seed(n)
    A = (torch.rand(n, n, generator=gen, device="cuda", dtype=dtype) - 0.5) * (2.0 / n)
    A.diagonal().fill_(1.0)
    X = torch.rand(n, nrhs, generator=gen, device="cuda", dtype=dtype) - 0.5
    LU, B = A.clone(), (A.double() @ X.double()).to(dtype)
    info = ebv.lu_factor_solve_(LU, B)
    assert int(info.item()) == 0
    eps = torch.finfo(dtype).eps
    # kappa <= 3: the solution to n eps times a few
    assert float((B.double() - X.double()).abs().max()) <= 4 * n * eps
    L = torch.tril(LU, -1).double()
    L.diagonal().fill_(1.0)
    assert float((L @ torch.triu(LU).double() - A.double()).abs().max()) <= n * eps
