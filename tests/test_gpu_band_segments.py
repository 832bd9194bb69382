"""GPU parity: the band factor and substitutions in segments (checked starts,
repeated where they disagree) against the oracle and the one-workgroup chain."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
from paper_1907_05767_amd import ebv, inputs
from tests.gpu_util import case, dev, fwd_err, host

pytestmark = pytest.mark.gpu


def _mask(n, kl, ku):
    j = np.arange(n)[:, None] + np.arange(kl + ku + 1)[None, :] - kl
    return (j >= 0) & (j < n)


def _run(AB, kl, ku, B, ws=None):
    t, X = dev(AB), dev(B)
    info = ebv.lu_factor_band_(t, kl, ku, ws=ws)
    ebv.lu_solve_band_(t, kl, ku, X)
    torch.cuda.synchronize()
    return host(t), host(X), int(info.item())


def _serial_ws():
    """A workspace too small for the segments: the one-workgroup chain."""
    return torch.empty(512, dtype=torch.uint8, device="cuda")


# 15 | 16 block rows: chain | segments of the factor; 47 | 48: of the sweeps;
# whole and partial last tiles and last segments, every chunking of the columns
@pytest.mark.parametrize("n,kl,ku,nrhs", [(960, 64, 64, 1), (961, 64, 64, 2), (1024, 3, 64, 16), (1100, 64, 0, 17),
                                          (3008, 64, 64, 33), (3009, 1, 2, 1), (3072, 64, 64, 40), (3200, 0, 0, 3),
                                          (5000, 33, 64, 16), (6147, 64, 31, 5)])
def test_band_segments_parity(n, kl, ku, nrhs):
    case(f"band segments n={n} kl={kl} ku={ku} nrhs={nrhs}")
    AB, B = inputs.band(n, kl, ku, 0.9, n), inputs.rhs(n, nrhs, n + 1)
    LU_ref, _ = oracle.lu_factor_band(AB, kl, ku)
    X_ref = oracle.lu_solve_band(LU_ref, kl, ku, B)
    LU, X, info = _run(AB, kl, ku, B)
    LU1, X1, _ = _run(AB, kl, ku, B, _serial_ws())
    m = _mask(n, kl, ku)
    assert info == 0
    assert np.abs(np.where(m, LU - LU_ref, 0)).max() <= 1e-12
    assert np.abs(np.where(m, LU1 - LU_ref, 0)).max() <= 1e-12
    assert fwd_err(X, X_ref) <= 1e-12 and fwd_err(X1, X_ref) <= 1e-12


def _grid(n):
    """Five-point Laplacian on a grid 64 wide: a chain that forgets slowly
    (about 0.9 per block row), so no segment's early start is good enough."""
    AB = np.zeros((n, 129))
    i = np.arange(n)
    AB[:, 64] = 4.0
    AB[i >= 64, 0] = -1.0
    AB[i < n - 64, 128] = -1.0
    AB[i % 64 != 0, 63] = -1.0
    AB[(i % 64 != 63) & (i < n - 1), 65] = -1.0
    return AB


@pytest.mark.parametrize("n", [1024, 3136])
def test_band_segments_repeated_where_they_disagree(n):
    case(f"band segments, slow decay n={n}")
    AB, B = _grid(n), inputs.rhs(n, 3, 7)
    LU_ref, _ = oracle.lu_factor_band(AB, 64, 64)
    X_ref = oracle.lu_solve_band(LU_ref, 64, 64, B)
    LU, X, info = _run(AB, 64, 64, B)
    assert info == 0
    # pivots within 1..4 and multipliers below 1: no growth; kappa below
    # 8 / (2 - 2 cos(pi / 65)) = 3.5e3, times eps times a small factor
    assert np.abs(np.where(_mask(n, 64, 64), LU - LU_ref, 0)).max() <= 1e-12
    assert fwd_err(X, X_ref) <= 1e-11


@pytest.mark.parametrize("cols", [(0,), (700,)])
def test_band_sweep_local_right_hand_side(cols):
    """A right-hand side in one row: the solution decays over the segments and
    keeps its relative accuracy block by block."""
    n = 3200
    case(f"band segments, local right-hand side {cols}")
    AB, B = inputs.band(n, 64, 64, 0.9, 5), np.zeros((n, 1))
    B[list(cols)] = 1.0
    LU_ref, _ = oracle.lu_factor_band(AB, 64, 64)
    X_ref = oracle.lu_solve_band(LU_ref, 64, 64, B)
    _, X, _ = _run(AB, 64, 64, B)
    blocks = np.arange(0, n, 64)
    err = np.maximum.reduceat(np.abs(X - X_ref)[:, 0], blocks) / np.maximum.reduceat(np.abs(X_ref)[:, 0], blocks)
    # each block's values are products of at most 50 contractions, each with a
    # relative error of a few 64 eps
    assert err.max() <= 50 * 64 * 4 * 2.2e-16


@pytest.mark.parametrize("rows", [(5,), (1400,), (2047, 900), (4,)])
def test_band_segments_zero_pivot(rows):
    """A row and column that meet nothing, with a zero diagonal: the first one
    is reported, also where it lies in a later segment."""
    n = 2048
    case(f"band segments zero pivots {rows}")
    AB = inputs.band(n, 64, 64, 0.5, 6)
    for r in rows:
        AB[r, :] = 0.0
        for d in range(-64, 65):
            if 0 <= r + d < n:
                AB[r + d, 64 - d] = 0.0
    _, info_ref = oracle.lu_factor_band(AB, 64, 64)
    t = dev(AB)
    info = ebv.lu_factor_band_(t, 64, 64)
    torch.cuda.synchronize()
    assert int(info.item()) == info_ref == min(rows) + 1


def _two_scales(n, c, couple, even=0.1):
    """Even and odd unknowns coupled to their like 64 away, the odd ones more
    strongly (and with `couple` to the even one before them): dominant, and
    slow enough to forget that the segments' starts differ from the chain."""
    i = np.arange(n)
    odd = i % 2 == 1
    AB = np.zeros((n, 129))
    AB[:, 64] = 1.0
    o = np.where(odd, -c, -even)
    AB[i >= 64, 0] = o[i >= 64]
    AB[i < n - 64, 128] = o[i < n - 64]
    AB[odd, 63] = couple
    return AB


def _times(AB, X):
    n, Y = len(AB), np.zeros_like(X)
    for d in range(129):
        lo, hi = max(0, 64 - d), min(n, n + 64 - d)
        Y[lo:hi] += AB[lo:hi, d:d + 1] * X[lo + d - 64:hi + d - 64]
    return Y


@pytest.mark.parametrize("c,scale", [(0.35, 1e-10), (0.25, 1e-8), (0.45, 1e-14), (0.25, 1e8), (0.35, 1.0)])
@pytest.mark.parametrize("what", ["rows", "unknowns"])
def test_band_sweep_of_two_scales(what, c, scale):
    """Rows, or the unknowns themselves, of two scales within every block: the
    small ones are as accurate as the large ones (kappa of either half <= 10)."""
    n = 4096
    case(f"band sweep two scales {what} c={c} scale={scale}")
    AB, X0 = _two_scales(n, c, 0.05 if what == "rows" else 0.0), inputs.rhs(n, 2, 3)
    if what == "rows":
        AB[1::2] *= scale
    else:
        X0[1::2] *= scale
    B = _times(AB, X0)
    LU_ref, _ = oracle.lu_factor_band(AB, 64, 64)
    X_ref = oracle.lu_solve_band(LU_ref, 64, 64, B)
    _, X, info = _run(AB, 64, 64, B)
    assert info == 0
    for half in (slice(0, None, 2), slice(1, None, 2)):
        assert fwd_err(X[half], X_ref[half]) <= 1e-12


@pytest.mark.parametrize("c,scale", [(0.25, 1e-10), (0.35, 1e-12), (0.45, 1e-15), (0.25, 1e10), (0.35, 1.0)])
def test_band_factor_of_two_scales(c, scale):
    """Columns of two scales: the factors, scales taken off, are O(1) and as
    accurate in the small columns as in the large ones."""
    n = 4096
    case(f"band factor two scales c={c} scale={scale}")
    col = np.where(np.arange(n) % 2 == 1, scale, 1.0)
    j = np.clip(np.arange(n)[:, None] + np.arange(129)[None, :] - 64, 0, n - 1)
    AB = _two_scales(n, c, 0.0, 0.0)
    i = np.arange(n)
    AB[(i % 2 == 1) & (i % 64 != 63), 65] = 0.05  # a large element in every odd row, which the
    AB[i % 64 == 63, 63] = 0.05                   # elimination leaves alone
    AB *= col[j]
    LU_ref, _ = oracle.lu_factor_band(AB, 64, 64)
    t = dev(AB)
    info = ebv.lu_factor_band_(t, 64, 64)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    off = np.where(np.arange(129)[None, :] >= 64, 1.0 / col[j], 1.0)  # U carries the columns' scales, L does not
    diff = np.where(_mask(n, 64, 64), (host(t) - LU_ref) * off, 0)
    assert np.abs(diff).max() <= 1e-12


def test_band_segments_zero_pivot_by_cancellation():
    """A pivot that the chain forms as an exact zero, in the first block row of a
    later segment: reported with the segments too, whose starts agree with the
    chain's tiles only to the last bits.

    Row m opens the segment with nothing above its diagonal 1; row r = m + 1
    meets only it on the left, with 1/2.  So u_rr = a_rr - u_mr / 2 exactly,
    u_mr being an element of the segment's first tile."""
    n = 4096
    case("band segments, zero pivots by cancellation")
    for m in range(256, n, 256):
        r = m + 1
        AB = inputs.band(n, 64, 64, 0.9, 11)
        for k in range(m - 64, m):
            AB[k, 64 + m - k] = 0.0
        AB[r, :64] = 0.0
        AB[r, 63] = 0.5
        t = dev(AB)
        assert int(ebv.lu_factor_band_(t, 64, 64, ws=_serial_ws()).item()) == 0
        AB[r, 64] = float(t[m, 65].item()) / 2
        t1, t2 = dev(AB), dev(AB)
        assert int(ebv.lu_factor_band_(t1, 64, 64, ws=_serial_ws()).item()) == r + 1
        assert int(ebv.lu_factor_band_(t2, 64, 64).item()) == r + 1


def test_band_segments_zero_pivot_in_a_repeated_segment():
    """The same in a segment that is factored again, behind others whose starts
    were kept although their last bits differ: all of them are taken again."""
    n, m = 2048, 1536
    r = m + 1
    case("band segments, zero pivot in a repeated segment")
    AB = inputs.band(n, 64, 64, 0.9, 11)
    AB[1024:] = _grid(n)[1024:]
    for k in range(m - 64, m):
        AB[k, 64 + m - k] = 0.0
    AB[r, :64] = 0.0
    AB[r, 63] = AB[m, 64] / 2
    t = dev(AB)
    assert int(ebv.lu_factor_band_(t, 64, 64, ws=_serial_ws()).item()) == 0
    AB[r, 64] = float(t[m, 65].item()) / 2
    t1, t2 = dev(AB), dev(AB)
    assert int(ebv.lu_factor_band_(t1, 64, 64, ws=_serial_ws()).item()) == r + 1
    assert int(ebv.lu_factor_band_(t2, 64, 64).item()) == r + 1
    assert torch.equal(t1[:m], t2[:m])  # the chain's factor, bit for bit


@pytest.mark.parametrize("n", [65536, 65537, 140000])
def test_band_segments_longer_than_four_rows(n):
    """More than 1024 block rows: segments of more than four, at most 256 of them."""
    case(f"band segments n={n}")
    AB, B = inputs.band(n, 5, 9, 0.9, n), inputs.rhs(n, 2, n + 1)
    LU_ref, _ = oracle.lu_factor_band(AB, 5, 9)
    X_ref = oracle.lu_solve_band(LU_ref, 5, 9, B)
    t, X = dev(AB), dev(B)
    info = ebv.lu_factor_band_(t, 5, 9)
    ebv.lu_solve_band_(t, 5, 9, X)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    j = np.arange(n)[:, None] + np.arange(15)[None, :] - 5
    assert np.abs(np.where((j >= 0) & (j < n), host(t) - LU_ref, 0)).max() <= 1e-12
    assert fwd_err(host(X), X_ref) <= 1e-12
