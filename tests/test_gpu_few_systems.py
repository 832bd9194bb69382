"""GPU: a ragged batch of fewer systems than the chip has compute units runs them
side by side, a unit each."""
from __future__ import annotations

import pytest
import torch

from paper_1907_05767_amd import ebv
from tests.gpu_util import case

pytestmark = pytest.mark.gpu


def _ms(count, n, form):
    dtype = torch.float32 if form == "f32" else torch.float64
    gen = torch.Generator(device="cuda").manual_seed(n)
    A0 = (torch.rand((count, n, n), generator=gen, device="cuda", dtype=dtype) - 0.5) * (2.0 / n)
    A0.diagonal(dim1=1, dim2=2).fill_(1.0)
    B0 = torch.rand(count * n, generator=gen, device="cuda", dtype=dtype)
    A, B = A0.clone(), B0.clone()
    rb = ebv.uniform_ragged(count, n)
    dt = ebv.F32 if form == "f32" else ebv.F64
    ws = ebv.workspace(ebv.OP_BATCHED_MIXED if form == "mixed" else ebv.OP_BATCHED, dt, A.numel(), B.numel(), count)
    best = float("inf")
    for _ in range(6):
        A.copy_(A0)
        B.copy_(B0)
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        info, _ = ebv.factor_solve_batched_(rb, A.view(-1), B, mixed=form == "mixed", ws=ws)
        e1.record()
        e1.synchronize()
        assert int(info.abs().max().item()) == 0
        best = min(best, e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("form", ["f64", "f32", "mixed"])
def test_few_systems_take_a_unit_each(form):
    """200 systems of n = 768 against one: alone on its unit a system keeps its
    pace (up to what the others take of the memory's rate, a few per cent); two
    to a unit take 1.5 times as long, three 1.8 times."""
    case(f"few systems {form}")
    one, many = _ms(1, 768, form), _ms(200, 768, form)
    print(f"{form}: one {one:.3f} ms, 200 {many:.3f} ms")
    assert many <= 1.3 * one
