"""The merge of a row's partial lists when they are more than its workgroup
takes at once: the bound found on the first batch also filters the later ones."""
import pytest
import torch

import paper_1805_02867_amd as osm
from parity import best_us

pytestmark = pytest.mark.gpu

N, H, V = 64, 1024, 98304  # 768 chunks of 4 lists: 24576 keys a row at K = 8, 16384 at once


@pytest.fixture(scope="module")
def inputs():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need an MI355X; none is visible")
    g = torch.Generator(device="cuda").manual_seed(5)
    h = torch.randint(-4, 5, (N, H), generator=g, device="cuda").bfloat16() * 0.125
    w = torch.randint(-4, 5, (V, H), generator=g, device="cuda").bfloat16() * 0.0625
    return h, w


@pytest.mark.parametrize("K", [6, 7, 8])
def test_indices(inputs, K):
    h, w = inputs
    print(f"K={K}", flush=True)
    vals, idx = osm.proj_softmax_topk(h, w, K)
    v, i = osm.softmax_topk(osm.proj(h, w), K)  # (the sums are exact in binary32)
    assert torch.equal(idx, i)
    assert torch.allclose(vals, v, rtol=2e-5, atol=0)


def test_later_batches_are_filtered(inputs):
    """Two batches against one: unfiltered, the second one's keys all went
    through the lists (63.8 us at K = 8, 43.5 at K = 5; 48.4 with the bound)."""
    h, w = inputs
    print("timing", flush=True)
    five, eight = (best_us(lambda: osm.proj_softmax_topk(h, w, K)) for K in (5, 8))
    print(f"{five:.1f} us, {eight:.1f} us", flush=True)
    assert eight <= 1.3 * five
