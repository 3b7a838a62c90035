"""More sizes for the order and the gather: the order at the edges of a wave's
part of a tile (512 primitives) and with so many tiles that each run of the
scan takes its unrolled loop and a remainder."""
import pytest
import torch

import test_gpu_order as order

pytestmark = pytest.mark.gpu

gs = pytest.importorskip("paper_2601_16736_amd")


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("kind", ["uniform", "few"])
@pytest.mark.parametrize("n", [511, 512, 513, 65_536 + 511, 65_536 + 512, 65_536 + 513, 5_000_011])
def test_order_at_the_parts_of_a_tile(n, kind):
    order.test_order_is_the_stable_sort_of_the_codes(n, kind)
