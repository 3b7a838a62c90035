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


@pytest.mark.parametrize("n", [1, 65, 4097, 2 ** 20 + 3])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("bf16", [False, True])
def test_prune_and_append_rows_of_threes(n, offset, bf16):
    dims = (3, 9, 45, 6) if n < 2 ** 20 else (3, 9)
    k = n // 3 + 1
    r = synth.rng(n, offset)

    def array(rows, d, dtype):
        buf = torch.from_numpy(r.standard_normal(rows * d + offset, dtype=np.float32)).to("cuda").to(dtype)
        return buf[offset:].view(rows, d)

    mdt = torch.bfloat16 if bf16 else torch.float32

    def groups(rows):
        return [gs.Group(array(rows, d, torch.float32), None, array(rows, d, mdt), array(rows, d, mdt), 1e-3)
                for d in dims]

    src, dst = groups(n), groups(n + k)
    t_src = torch.arange(n, dtype=torch.int32, device="cuda")
    t_dst = torch.full((n + k,), -5, dtype=torch.int32, device="cuda")
    keep = torch.from_numpy((r.random(n) < 0.9).astype(np.uint8)).to("cuda")
    count = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(gs.gs_prune_workspace_size(n), dtype=torch.uint8, device="cuda")
    rows = torch.nonzero(keep)[:, 0]
    kept = int(rows.numel())
    pick = torch.from_numpy(r.integers(0, max(kept, 1), k).astype(np.int32)).to("cuda")
    arrays = [(a, b) for s, d in zip(src, dst) for a, b in ((s.param, d.param), (s.exp_avg, d.exp_avg),
                                                           (s.exp_avg_sq, d.exp_avg_sq))]
    after = [b[kept:].clone() for _, b in arrays]
    print(f"threes prune n={n} offset={offset} bf16={bf16}", flush=True)
    gs.gs_prune(keep, src, dst, int(bf16), t_src, t_dst, count, ws)
    torch.cuda.synchronize()
    assert int(count) == kept and torch.equal(t_dst[:kept], t_src[rows])
    for (a, b), rest in zip(arrays, after):
        assert torch.equal(b[:kept], a[rows]) and torch.equal(b[kept:], rest)
    if kept == 0:
        return
    gs.gs_append(dst, int(bf16), kept, pick, t_dst)
    torch.cuda.synchronize()
    for j, (a, b) in enumerate(arrays):
        new = torch.zeros_like(b[:k]) if j % 3 else a[rows][pick.long()]
        assert torch.equal(b[:kept], a[rows]) and torch.equal(b[kept:kept + k], new)
        assert torch.equal(b[kept + k:], after[j][k:])
