"""gs_gather_rows for every chunk width it chooses (16, 8, 4, 2 and 1 bytes,
and 12 for word-aligned rows that are multiples of it), at row counts around
its blocks, with misaligned arrays and out-of-range entries: dst row i is src
row perm[i] byte for byte, and rows with an entry outside [0, n) stay as they
were."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")
from _gpu_util import DEV  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("offset", [0, 4, 2, 1])
@pytest.mark.parametrize("row_bytes", [1, 2, 3, 4, 6, 8, 12, 16, 20, 24, 36, 90, 96, 180, 192, 4100, 16384])
def test_gather_rows_every_chunk_width(row_bytes, offset):
    for n in (1, 2, 21, 22, 255, 256, 257, 1031):
        r = synth.rng(row_bytes, offset, n)
        src = r.integers(0, 256, (n, row_bytes), dtype=np.uint8)
        dst = r.integers(0, 256, (n, row_bytes), dtype=np.uint8)
        perm = r.integers(0, n, n).astype(np.int32)
        perm[::7] = r.choice(np.array([-1, n, 2**31 - 1, -(2**31)], np.int64), perm[::7].size).astype(np.int32)
        guard = 32
        raw = [torch.zeros(offset + n * row_bytes + guard, dtype=torch.uint8, device=DEV) for _ in range(2)]
        views = [x[offset:offset + n * row_bytes].view(n, row_bytes) for x in raw]
        views[0].copy_(torch.from_numpy(src))
        views[1].copy_(torch.from_numpy(dst))
        print(f"gather n={n} row_bytes={row_bytes} offset={offset}", flush=True)
        gs.gs_gather_rows(views[0], views[1], torch.from_numpy(perm).to(DEV))
        torch.cuda.synchronize()
        ok = (perm >= 0) & (perm < n)
        want = dst.copy()
        want[ok] = src[perm[ok]]
        np.testing.assert_array_equal(views[1].cpu().numpy(), want)
        assert int(raw[1][:offset].sum()) == 0 and int(raw[1][offset + n * row_bytes:].sum()) == 0
