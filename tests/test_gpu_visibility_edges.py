"""gs_visibility_multi without a radius decides most points without a division;
every bit must still equal gs_visibility's (which divides) and the oracle's,
on points packed around the image edges (within a few units in the last place
of the projected coordinate), at tiny and huge depths, and on NaN, infinite
and overflowing means, for cameras whose edges lie at zero, at negative, odd
and large pixel coordinates."""
import itertools
import math

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")
from _gpu_util import DEV  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    oracle.build(force=False)


IDENTITY = [1, 0, 0, 0, 0, 1, 0, 0, 0, 0, 1, 0]


def _points(cam, n, seed):
    """Points whose projections crowd the four image edges of an axis camera,
    depths over many binades, and special values."""
    r = synth.rng(seed, n)
    z = np.exp2(r.uniform(-40, 40, n)).astype(np.float32)
    z[::5] = r.uniform(0.1, 30, z[::5].size).astype(np.float32)
    edges_x = r.choice(np.array([0.0, cam["width"], r.uniform(0, cam["width"])]), n)
    edges_y = r.choice(np.array([0.0, cam["height"], r.uniform(0, cam["height"])]), n)
    with np.errstate(over="ignore"):
        x = ((edges_x - cam["cx"]) * z.astype(np.float64) / cam["fx"]).astype(np.float32)
        y = ((edges_y - cam["cy"]) * z.astype(np.float64) / cam["fy"]).astype(np.float32)
    p = np.stack([x, y, z], 1)
    bits = p[:, :2].copy().view(np.int32)
    bits += r.integers(-3, 4, bits.shape, dtype=np.int32)      # a few units in the last place
    p[:, :2] = bits.view(np.float32)
    special = np.array([np.nan, np.inf, -np.inf, 3e38, -3e38, 1e-45, -1e-45, 0.0, -0.0, 1e-38], np.float32)
    rows = np.array(list(itertools.product(special, repeat=3)), np.float32)
    p[: min(n, len(rows))] = rows[: min(n, len(rows))]
    return np.ascontiguousarray(p)


CAMERAS = [dict(fx=500.0, fy=500.0, cx=500.0, cy=500.0, width=1000, height=1000),
           dict(fx=866.0254, fy=433.3, cx=0.0, cy=-37.25, width=1, height=4097),
           dict(fx=1.5e-3, fy=7e5, cx=333.333, cy=1e7, width=999, height=2**30),
           dict(fx=-250.0, fy=1e30, cx=2.0**70, cy=0.1, width=640, height=480),
           dict(fx=1e-30, fy=3.0, cx=-5e-40, cy=479.5, width=641, height=479)]


@pytest.mark.parametrize("n", [1, 1023, 4096, 4097, 50_021])
def test_multi_view_bits_equal_the_divided_predicate(n):
    cams = [gs.Camera(IDENTITY, c["fx"], c["fy"], c["cx"], c["cy"], c["width"], c["height"], 0.0, zf)
            for c in CAMERAS for zf in (math.inf, 17.5)]
    ocams = [oracle.Camera(np.array(IDENTITY, np.float32).reshape(3, 4), c["fx"], c["fy"], c["cx"], c["cy"], c["width"],
                           c["height"], 0.0, zf) for c in CAMERAS for zf in (math.inf, 17.5)]
    for k, c in enumerate(CAMERAS):
        pts = _points(c, n, 300 + k)
        means = torch.from_numpy(pts).to(DEV)
        bits = torch.zeros(n, dtype=torch.int32, device=DEV)
        union = torch.zeros(n, dtype=torch.uint8, device=DEV)
        gs.gs_visibility_multi(means, cams, mask=union, view_bits=bits)
        torch.cuda.synchronize()
        got = bits.cpu().numpy()
        for v, (cam, ocam) in enumerate(zip(cams, ocams)):
            one = torch.zeros(n, dtype=torch.uint8, device=DEV)
            gs.gs_visibility(means, cam, mask=one)
            np.testing.assert_array_equal((got >> v) & 1, one.cpu().numpy(), err_msg=f"points {k}, view {v}")
            with np.errstate(all="ignore"):
                np.testing.assert_array_equal((got >> v) & 1, oracle.visibility(pts, ocam), err_msg=f"oracle, view {v}")
        np.testing.assert_array_equal(union.cpu().numpy(), (got != 0).astype(np.uint8))
