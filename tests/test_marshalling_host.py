"""The packed structures hold the bytes that setting them field by field gives,
and both ways fail alike."""
import random

import numpy as np
import pytest
import torch

import paper_2601_16736_amd as gs


def _outcome(make):
    try:
        return bytes(make())
    except Exception as e:
        return type(e), str(e)


def _group(rng):
    n, d = rng.choice([0, 1, 5]), rng.choice([1, 3, 48])
    kinds = [lambda: torch.zeros(n, d), lambda: torch.nn.Parameter(torch.zeros(n, d)),
             lambda: torch.zeros(n, 64)[:, :d], lambda: torch.zeros(d, n).t(), lambda: torch.zeros(n, 2 * d)[:, ::2],
             lambda: torch.zeros(n), lambda: torch.zeros(n, d, 2), lambda: 4096]
    if rng.random() < 0.5:
        kinds = [rng.choice(kinds)]
    p, g, m, v = (rng.choice(kinds)() for _ in range(4))
    return gs.Group(p, rng.choice([g, None]), m, v, rng.choice([1e-3, 1, "0.5", torch.tensor(2.0)]),
                    rng.choice([0, 1, 1.0, 2 ** 40]), 0.1, rng.choice([10.0, float("inf")]), rng.choice([0, 1]),
                    rng.choice([None, None, None, 64]))


def _camera(rng):
    v = [rng.gauss(0, 1) for _ in range(rng.choice([12, 12, 12, 11, 13]))]
    views = [v, tuple(v), np.array(v), torch.tensor(v, dtype=torch.float64), [str(x) for x in v], [1] * 12, None]
    if len(v) == 12:
        views += [np.array(v, np.float32).reshape(3, 4), torch.tensor(v).reshape(3, 4), torch.tensor(v).reshape(4, 3).t()]
    return gs.Camera(rng.choice(views), rng.choice([500.0, 5, 1e39, float("nan")]), 400.0, 3.0, 4.0,
                     rng.choice([640, 640.0, "640", "x", 2 ** 33]), 480, 0.1, rng.choice([100.0, float("inf"), 1e40]), 0.5)


def _config(rng):
    return gs.StepConfig(beta1=rng.choice([0.9, 0, "0.9"]), seed=rng.choice([0, -1, 2 ** 70, 7.0]),
                         iteration=rng.choice([0, 5, 2 ** 40, 2 ** 70]), moment_dtype=rng.choice([0, 1, True]),
                         stochastic_round=rng.choice([True, False, 0]), rsr_enable=rng.random() < 0.5,
                         schedule=rng.randrange(5), rsr_ratio=rng.random(), visible_hint=rng.choice([0.2, "0.2"]),
                         unit=rng.choice([0, 64, 2 ** 33 + 5]), noise_enable=rng.random() < 0.5,
                         noise_groups=rng.choice([(0, 1, 2, 3), [3, 2, 1, 0], (0, 1)]), noise_lr=rng.random(),
                         aiu_enable=rng.random() < 0.5, aiu_ratio=rng.random(), aiu_scale=1)


@pytest.mark.parametrize("make", [_group, _camera, _config])
def test_packed_equals_field_by_field(make):
    rng = random.Random(5)
    for _ in range(500):
        x = make(rng)
        assert _outcome(x.to_c) == _outcome(x._by_field), x
