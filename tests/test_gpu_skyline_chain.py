"""GPU parity of the skyline factor and its chained substitutions at their edges: block counts
around the number of dependencies a block treats apart (the last two in
registers, the third polled, older ones shared with the helper), empty and
far-apart dependencies, one to several chunks of 16 right-hand sides, and
solves repeated on one set of factors, against the skyline oracle.

The tolerance is the one of the other skyline tests (relative 1e-12 on
diagonally dominant systems)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, fwd_err, host

pytestmark = pytest.mark.gpu


def _profile(kind: str, n: int, rng) -> tuple[np.ndarray, np.ndarray]:
    idx = np.arange(n)
    if kind == "full":
        return np.zeros(n, np.int32), np.zeros(n, np.int32)
    if kind == "diagonal":
        return idx.astype(np.int32), idx.astype(np.int32)
    if kind == "lower":  # full lower part, diagonal upper part
        return np.zeros(n, np.int32), idx.astype(np.int32)
    # "spikes": narrow rows and columns with a few that reach far back, so that
    # a block's upper dependencies are not adjacent blocks
    f, g = np.maximum(idx - 3, 0), np.maximum(idx - 5, 0)
    for v in (f, g):
        far = rng.choice(n, size=max(1, n // 90), replace=False)
        v[far] = (v[far] * rng.random(far.size)).astype(np.int64)
    return f.astype(np.int32), g.astype(np.int32)


def _system(kind: str, n: int, seed: int):
    f, g = _profile(kind, n, np.random.default_rng(seed))
    idx = np.arange(n)
    rp, cp = np.zeros(n + 1, np.int64), np.zeros(n + 1, np.int64)
    rp[1:], cp[1:] = np.cumsum(idx - f), np.cumsum(idx - g + 1)
    A = inputs.dense(n, 0.5, seed)
    AL = np.concatenate([A[i, f[i]:i] for i in range(n)])
    AU = np.concatenate([A[g[j]:j + 1, j] for j in range(n)])
    return f, rp, AL, g, cp, AU


@pytest.mark.parametrize("kind,n,nrhs", [
    ("full", 1, 1), ("full", 64, 16), ("full", 65, 17), ("full", 128, 1), ("full", 129, 8), ("full", 192, 16),
    ("full", 250, 40), ("full", 257, 2), ("full", 321, 16), ("full", 449, 33), ("full", 1000, 5),
    ("diagonal", 130, 3), ("diagonal", 640, 17), ("lower", 400, 16), ("spikes", 500, 1), ("spikes", 1500, 20),
    ("spikes", 2049, 9),
])
def test_skyline_chain(kind, n, nrhs):
    case(f"skyline chain {kind} n={n} nrhs={nrhs}")
    f, rp, AL, g, cp, AU = _system(kind, n, 1700 + n)
    LL, UU, info = oracle.lu_factor_skyline(f, rp, AL, g, cp, AU)
    assert info == 0
    sk = ebv.Skyline(f, rp, AL, g, cp, AU)
    assert int(sk.factor_().item()) == 0
    for rep in range(2):
        B = inputs.rhs(n, nrhs, 1700 + n + rep)
        buf = torch.full((n + 2, nrhs), 7.25, dtype=torch.float64, device="cuda")
        buf[1:n + 1] = torch.from_numpy(B).cuda()
        sk.solve_(buf[1:n + 1])
        torch.cuda.synchronize()
        assert fwd_err(host(buf[1:n + 1]), oracle.lu_solve_skyline(f, rp, LL, g, cp, UU, B)) <= 1e-12
        assert bool((buf[0] == 7.25).all()) and bool((buf[n + 1] == 7.25).all())


def test_skyline_first_zero_pivot():
    """Independent diagonal tiles finish in any order: the smallest zero pivot is reported."""
    case("skyline first zero pivot")
    f, rp, AL, g, cp, AU = _system("diagonal", 1000, 5)
    for i in (900, 333, 70):
        AU[i] = 0.0
    sk = ebv.Skyline(f, rp, AL, g, cp, AU)
    assert int(sk.factor_().item()) == 71
    assert oracle.lu_factor_skyline(f, rp, AL, g, cp, AU)[2] == 71
