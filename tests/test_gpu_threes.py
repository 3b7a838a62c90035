"""Rows of three, nine, fifteen and 45 elements, which move three at a time,
against the oracle: isolated and all rows visible (the two sides of the hint's
rule), remainders of trips, odd offsets and odd rows of BF16 pairs, with Re-State."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_shapes as shapes

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("visible", [0.3, 0.9, 1.0])
@pytest.mark.parametrize("dims,offsets", [((3, 9, 45), None), ((15, 3, 21), [1, 2, 3]), ((45, 3, 1), [3, 1, 0])])
@pytest.mark.parametrize("sched,unit", [(gs.GS_SCHED_COMPACTED, 64), (gs.GS_SCHED_MASKED, 32),
                                        (gs.GS_SCHED_MASKED, 256)])
@pytest.mark.parametrize("bf16", [False, True])
def test_step_of_rows_of_threes(dims, offsets, sched, unit, bf16, visible, monkeypatch):
    monkeypatch.setattr(synth, "bernoulli_mask",
                        lambda n, p, *key: (synth.rng(3, n).random(n) < visible).astype(np.uint8))
    for n in (1, 33, 1501):
        shapes._run(n, dims, sched, unit, bf16, seed=n, offsets=offsets)
