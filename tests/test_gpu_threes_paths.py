"""The paths of rows of threes that depend on what else a call holds: the
fused view step with rows of 45 elements, over isolated visible rows and over
runs of them, and the instances of the batched plan (with and without groups
that go three elements at a time, with and without packed rows), each bit for
bit what the two-launch step gives."""
import numpy as np
import pytest
import torch

import synth
import test_gpu_packed as packed
import test_gpu_view as view
from test_gpu_layout import morton_codes_host

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")
from _gpu_util import DEV, make_state  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("ordered", [False, True])
@pytest.mark.parametrize("unit,bf16,noise", [(32, False, False), (32, True, False), (64, True, True),
                                             (128, False, True), (256, True, False)])
def test_view_step_with_wide_rows_of_threes(unit, bf16, noise, ordered, monkeypatch):
    monkeypatch.setattr(synth, "GROUPS_59", synth.GROUPS_60_SPLIT)
    scene = view._scene

    def arranged(n, seed, bf16):
        st = scene(n, seed, bf16)
        if ordered:
            m = st.groups[0].param
            at = np.argsort(morton_codes_host(m.cpu().numpy()), kind="stable")
            m.copy_(m[torch.from_numpy(at).to(DEV)].clone())
        return st

    monkeypatch.setattr(view, "_scene", arranged)
    for n in (33, 20_011):
        view.test_view_step_equals_visibility_then_step(n, unit, bf16, True, True, noise, False)


def _flat(n, spec, seed, bf16):
    st = make_state(gs, n, spec, seed, bf16=bf16)
    for k, g in enumerate(st.groups):
        g.grad.copy_(torch.from_numpy(1e-3 * synth.rng(seed, k).standard_normal(tuple(g.grad.shape), dtype=np.float32)))
    return st.groups, st.t, *view._clone(st)


@pytest.mark.parametrize("kinds", [("59",), ("60",), ("packed",), ("packed", "59", "60")])
@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("noise", [False, True])
def test_batched_plan_instances(kinds, bf16, noise):
    specs = {"59": synth.GROUPS_59, "60": synth.GROUPS_60_SPLIT}
    scenes, refs, twins = [], [], []
    for s, kind in enumerate(kinds):
        n = (5003, 257, 1501)[s]
        if kind == "packed":
            tw = packed.Twin(n, 61 + s, bf16)
            twins.append(tw)
            groups, t, ref, ref_t = tw.packed, tw.t_pack, tw.flat, tw.t_flat
        else:
            groups, t, ref, ref_t = _flat(n, specs[kind], 71 + s, bf16)
        mask = torch.from_numpy(synth.bernoulli_mask(n, 0.4, 5, s)).to(DEV)
        scenes.append(gs.Scene(groups=groups, n=n, step_count=t, visible=mask, schedule=gs.GS_SCHED_MASKED))
        refs.append((groups, t, ref, ref_t, mask, n))
    batch = gs.Batch(scenes, moment_dtype=int(bf16))
    print(f"plan {kinds} bf16={bf16} noise={noise}", flush=True)
    for it in range(3):
        kw = dict(iteration=it, moment_dtype=int(bf16), rsr_enable=it == 1, rsr_ratio=0.3, aiu_enable=it == 2,
                  aiu_ratio=0.4, aiu_scale=0.5, noise_enable=noise, noise_lr=300.0, noise_t=0.5)
        batch.step(gs.StepConfig(seed=9, **kw))
        for s, (groups, t, ref, ref_t, mask, n) in enumerate(refs):
            gs.adamw_gs_step(ref, n, ref_t, gs.StepConfig(seed=9 + s, schedule=gs.GS_SCHED_MASKED, **kw), visible=mask)
    torch.cuda.synchronize()
    for tw in twins:
        tw.check_same("plan")
    for groups, t, ref, ref_t, _, _ in refs:
        assert torch.equal(t, ref_t)
        for a, b in zip(groups, ref):
            for x, y in ((a.param, b.param), (a.exp_avg, b.exp_avg), (a.exp_avg_sq, b.exp_avg_sq)):
                assert torch.equal(view._bits(x.contiguous()), view._bits(y.contiguous()))
    batch.close()
