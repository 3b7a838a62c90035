"""More sizes for the order and the gather: the order at the edges of a wave's
part of a tile (512 primitives) and with so many tiles that each run of the
scan takes its unrolled loop and a remainder; the gather on both sides of its
longest rows (2^22 chunks), in chunks of one, two and twelve bytes."""
import pytest
import torch

import test_gpu_order as order

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")
from _gpu_util import DEV  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("kind", ["uniform", "few"])
@pytest.mark.parametrize("n", [511, 512, 513, 65_536 + 511, 65_536 + 512, 65_536 + 513, 5_000_011])
def test_order_at_the_parts_of_a_tile(n, kind):
    order.test_order_is_the_stable_sort_of_the_codes(n, kind)


@pytest.mark.parametrize("chunks", [2 ** 22 - 1, 2 ** 22, 2 ** 22 + 1])
@pytest.mark.parametrize("width,offset", [(1, 1), (2, 2), (12, 4)])
def test_gather_of_the_longest_rows(chunks, width, offset):
    n, row = 3, chunks * width
    g = torch.Generator(device=DEV)
    g.manual_seed(chunks + width)
    raw = [torch.randint(0, 256, (offset + n * row + 32,), generator=g, device=DEV, dtype=torch.uint8) for _ in range(2)]
    src, dst = (x[offset:offset + n * row].view(n, row) for x in raw)
    before = raw[1].clone()
    print(f"gather row_bytes={row} offset={offset}", flush=True)
    gs.gs_gather_rows(src, dst, torch.tensor([2, -1, 0], dtype=torch.int32, device=DEV))
    torch.cuda.synchronize()
    was = before[offset:offset + n * row].view(n, row)
    assert torch.equal(dst[0], src[2]) and torch.equal(dst[1], was[1]) and torch.equal(dst[2], src[0])
    assert torch.equal(raw[1][:offset], before[:offset]) and torch.equal(raw[1][offset + n * row:], before[offset + n * row:])
