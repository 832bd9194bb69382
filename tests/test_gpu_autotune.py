"""GPU: the autotuner's dense sweeps vary settings that act on the calls they time."""
from __future__ import annotations

import pytest
import torch

from paper_1907_05767_amd import autotune, ebv, inputs
from tests.gpu_util import case

pytestmark = pytest.mark.gpu


def test_dense_sweep_runs_block_steps():
    case("autotuner: dense sweep")
    results, best = autotune.sweep_dense(torch, ebv, inputs, 1, (1, 3), (512,), n=1500, nrhs=2400)
    assert [r["defer_group"] for r in results] == [1, 3] and best in results


def test_dense_sweep_refuses_one_launch():
    """A call that runs as one launch has nothing to vary."""
    case("autotuner: dense sweep of a one-launch factor")
    with pytest.raises(SystemExit):
        autotune.sweep_dense(torch, ebv, inputs, 1, (1,), (512,), n=300, nrhs=8)
