"""gs_spatial_order at the edges of its tiles (4096 primitives, 512 to a wave)
and digits: the stable order of the host's Morton codes, exactly; eagerly and
from a captured graph replayed on other means."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")
from _gpu_util import DEV  # noqa: E402
from test_gpu_layout import morton_codes_host  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _means(n, kind, seed):
    r = synth.rng(seed, n)
    m = r.uniform(-3, 3, (n, 3)).astype(np.float32)
    if kind == "few":                   # long ties
        m = r.integers(0, 3, (n, 3)).astype(np.float32)
    if kind == "one":
        m[:] = m[0]
    if kind == "line":                  # one axis has no extent, the codes descend
        m[:, 1] = 2.0
        m[:, 0] = m[:, 2] = -np.arange(n, dtype=np.float32)
    if kind == "nan":
        m[r.random((n, 3)) < 0.2] = np.nan
        m[0], m[-1] = 0.0, 1.0
    return m


@pytest.mark.parametrize("kind", ["uniform", "few", "one", "line", "nan"])
@pytest.mark.parametrize("n", [1, 2, 63, 65, 1023, 1025, 4095, 4096, 4097, 8193, 65_535, 65_536, 70_001, 270_337])
def test_order_is_the_stable_sort_of_the_codes(n, kind):
    perm = torch.full((n + 1,), -7, dtype=torch.int32, device=DEV)
    size = gs.gs_spatial_order_workspace_size(n)
    ws = torch.full((size + 256,), 0xA5, dtype=torch.uint8, device=DEV)
    means = torch.zeros(n, 3, device=DEV)

    def check(m):
        want = np.argsort(morton_codes_host(m), kind="stable")
        torch.cuda.synchronize()
        np.testing.assert_array_equal(perm[:n].cpu().numpy(), want)
        assert int(perm[n]) == -7 and bool((ws[size:] == 0xA5).all())
        perm[:n] = -1

    m = _means(n, kind, 1)
    means.copy_(torch.from_numpy(m))
    gs.gs_spatial_order(means, perm[:n], ws[:size])
    check(m)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gs.gs_spatial_order(means, perm[:n], ws[:size])
    for seed in (2, 3):
        m = _means(n, kind, seed)
        means.copy_(torch.from_numpy(m))
        graph.replay()
        check(m)
