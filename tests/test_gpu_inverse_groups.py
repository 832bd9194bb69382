"""GPU parity: the explicit inverse where its tiles take the terms of several
block steps at once -- every remainder of the groups, partial last blocks, and
launches below and above the size at which whole tiles are used."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [257, 320, 385, 447, 577, 1000, 2625])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_inverse_groups(n, dtype):
    case(f"inverse groups n={n} {dtype}")
    A = inputs.dense(n, 0.5, 40 + n)
    LU, info = ebv.lu_factor(dev(A, dtype))
    pitch = n + 5  # the result's own leading dimension, its gap untouched
    out = torch.full((n, pitch), 3.0, dtype=dtype, device="cuda")
    dt = ebv.F64 if dtype == torch.float64 else ebv.F32
    w, wb = ebv._ws_args(ebv.workspace(ebv.OP_INVERSE, dt, n, 0))
    rc = ebv.lib().ebv_lu_inverse(ebv.handle(), dt, n, ebv._p(LU), n, ebv._p(out), pitch, w, wb, ebv._stream())
    torch.cuda.synchronize()
    assert rc == 0 and int(info.item()) == 0
    assert bool((out[:, n:] == 3.0).all())
    X = host(out[:, :n]).astype(np.float64)
    # kappa <= 3 in the maximum norm, entries of the inverse at most 2: A X
    # differs from I by a few n eps
    eps = 2.2e-16 if dtype == torch.float64 else 1.2e-7
    assert np.abs(A @ X - np.eye(n)).max() <= 4 * n * eps


@pytest.mark.parametrize("n", [2047, 2048, 2049, 3072, 3073, 3137, 3201, 3265, 3330, 6144, 6145])
def test_inverse_groups_by_size(n):
    """The sizes at which a tile takes one, two or four block steps at a time, and
    every remainder of the four (the residual formed on the device in FP64)."""
    case(f"inverse group sizes n={n}")
    A = dev(inputs.dense(n, 0.5, 40 + n))
    for dtype, eps in ((torch.float64, 2.2e-16), (torch.float32, 1.2e-7)):
        LU, info = ebv.lu_factor(A.to(dtype))
        X = ebv.lu_inverse(LU).double()
        assert int(info.item()) == 0
        R = A @ X
        R.diagonal().sub_(1.0)
        assert float(R.abs().max()) <= 4 * n * eps
