"""GPU parity: ragged batches in FP32 and in mixed precision with two and with
three workgroups to a compute unit (chosen by the number of systems), at the sizes
where the mixed form's solution vector moves: LDS up to n = 4160, or with three to a unit up
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


@pytest.mark.parametrize("count", [2, 513, 600, 1025, 1537])
@pytest.mark.parametrize("even", [False, True])
@pytest.mark.parametrize("form", ["f32", "mixed"])
def test_forms_on_both_sides_of_the_dispatch(form, even, count):
    case(f"ragged forms {form} even={even} count={count}")
    kinds = [40, 40] if even else [17, 130]
    ns = np.array([kinds[i % 2] for i in range(count)], dtype=np.int32)
    As = {m: inputs.dense(m, 0.5, m) for m in set(kinds)}
    Bs = {m: inputs.rhs(m, 1, m + 1) for m in set(kinds)}
    dt = torch.float32 if form == "f32" else torch.float64
    A = dev(np.concatenate([As[int(m)].ravel() for m in ns]), dt)
    B = dev(np.concatenate([Bs[int(m)].ravel() for m in ns]), dt)
    offA = np.concatenate([[0], np.cumsum(ns.astype(np.int64) ** 2)[:-1]])
    offB = np.concatenate([[0], np.cumsum(ns.astype(np.int64))[:-1]])
    info, _ = ebv.factor_solve_batched_(ebv.RaggedBatch(ns, offA, offB), A, B, mixed=form == "mixed")
    torch.cuda.synchronize()
    assert int(info.abs().max().item()) == 0
    X = host(B).astype(np.float64)
    # kappa <= 3 and n eps per solve, with a margin of 4 in FP32
    tol = 1e-12 if form == "mixed" else 4 * 130 * 6e-8
    for m in set(kinds):
        ref = oracle.solve(As[m], Bs[m])[0][:, 0]
        got = np.stack([X[o:o + m] for o, k in zip(offB, ns) if k == m])
        assert np.abs(got - ref).max() <= tol * np.abs(ref).max()
