"""GPU parity: the mixed-precision ragged batch with two and with three
workgroups to a compute unit (chosen by the number of systems), at the sizes
where its solution vector moves: LDS up to n = 4160, or with three to a unit up
to 1568 and memory beyond.

Dominant systems with row sum 0.5: the refinement stops at a relative error
bound of 1e-12."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, fwd_err, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1567, 1568, 1569, 2100, 4160, 4161])
@pytest.mark.parametrize("three", [False, True])
def test_mixed_vector_in_lds_and_memory(n, three):
    case(f"mixed batch forms n={n} three to a unit={three}")
    # more than six systems a unit: three workgroups to a unit, else two
    units = torch.cuda.get_device_properties(0).multi_processor_count
    m = 24
    small = 6 * units + 1 if three else 1
    ns = np.array([n] + [m] * small, dtype=np.int32)
    As = [inputs.dense(n, 0.5, n), inputs.dense(m, 0.5, 5)]
    Bs = [inputs.rhs(n, 1, n + 1), inputs.rhs(m, 1, 6)]
    A = dev(np.concatenate([As[0].ravel()] + [As[1].ravel()] * small))
    B = dev(np.concatenate([Bs[0].ravel()] + [Bs[1].ravel()] * small))
    offA = np.concatenate([[0], np.cumsum(ns.astype(np.int64) ** 2)[:-1]])
    offB = np.concatenate([[0], np.cumsum(ns.astype(np.int64))[:-1]])
    before = A.clone()
    info, iters = ebv.factor_solve_batched_(ebv.RaggedBatch(ns, offA, offB), A, B, mixed=True)
    torch.cuda.synchronize()
    assert int(info.abs().max().item()) == 0
    assert int(iters.min().item()) >= 0 and int(iters.max().item()) <= 3
    assert torch.equal(A, before)
    X = host(B)
    assert fwd_err(X[:n][:, None], oracle.solve(As[0], Bs[0])[0]) <= 1e-12
    ref = oracle.solve(As[1], Bs[1])[0]
    assert np.abs(X[n:].reshape(small, m) - ref[:, 0]).max() <= 1e-12 * np.abs(ref).max()
