"""GPU parity: one-workgroup systems at the edges of their tile pieces -- two
tiles at a time, a last single one, partial ones in both directions -- and the
mixed-precision form on both sides of the sizes its vectors fit LDS."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, fwd_err, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 320, 449])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_batched_pieces(n, dtype):
    case(f"batched pieces n={n} {dtype}")
    ns = [n, max(1, n - 1), n]
    As = [inputs.dense(m, 0.5, 70 + m + i) for i, m in enumerate(ns)]
    Bs = [inputs.rhs(m, 1, 80 + m + i) for i, m in enumerate(ns)]
    if dtype == torch.float32:
        As, Bs = ([x.astype(np.float32).astype(np.float64) for x in v] for v in (As, Bs))
    offA = np.concatenate([[0], np.cumsum([m * m for m in ns])[:-1]])
    offB = np.concatenate([[0], np.cumsum(ns)[:-1]])
    A = dev(np.concatenate([a.ravel() for a in As]), dtype)
    B = dev(np.concatenate([b.ravel() for b in Bs]), dtype)
    rb = ebv.RaggedBatch(ns, offA, offB)
    info, _ = ebv.factor_solve_batched_(rb, A, B)
    U = dev(np.stack([As[0], As[2]]), dtype)  # the uniform form, factor only
    ebv.lu_factor_(U)
    torch.cuda.synchronize()
    tol = 1e-12 if dtype == torch.float64 else 4 * n * 6e-8 + 1e-6
    assert host(info).tolist() == [0, 0, 0]
    for k, m in enumerate(ns):
        X_ref, LU_ref, _ = oracle.solve(As[k], Bs[k])
        LU = host(A[offA[k]:offA[k] + m * m]).reshape(m, m)
        assert np.abs(LU - LU_ref).max() <= tol
        assert fwd_err(host(B[offB[k]:offB[k] + m])[:, None], X_ref) <= tol
        if k != 1:
            assert np.abs(host(U[k // 2]) - LU_ref).max() <= tol


@pytest.mark.parametrize("n", [1311, 1312, 1313])
def test_batched_mixed_vector_places(n):
    case(f"batched mixed n={n}")
    A, B = inputs.dense(n, 0.5, n), inputs.rhs(n, 1, n + 1)
    X_ref, _, _ = oracle.solve(A, B)
    tA, tB = dev(A).view(-1), dev(B).view(-1)
    rb = ebv.RaggedBatch([n], [0], [0])
    info, iters = ebv.factor_solve_batched_(rb, tA, tB, mixed=True)
    torch.cuda.synchronize()
    assert int(info.item()) == 0 and 0 <= int(iters.item()) <= 3
    assert np.array_equal(host(tA).reshape(n, n), A)
    assert fwd_err(host(tB)[:, None], X_ref) <= 1e-12
