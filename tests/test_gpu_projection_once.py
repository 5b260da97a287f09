"""One strip of batch rows against a vocabulary of 384 MiB and more, whose rows
are then loaded with the non-temporal policy: the same bits as slices of the
vocabulary below that size give, and top-k of them exact."""
import pytest
import torch

import paper_1805_02867_amd as osm
from parity import RTOL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K,H,V", [
    (1, 5, 4096, 49153), (64, 16, 4096, 49153),  # 384 MiB and one row of 8 KiB
    (100, 5, 4096, 49153), (128, 16, 4096, 49153), (200, 8, 4096, 49153),
    (256, 12, 2048, 98305),                      # lists of 16 in one strip of 256
    (256, 12, 4096, 49153),                      # in two strips of 128: the default policy
    (64, 5, 4088, 49300), (64, 12, 4104, 49300),  # rows of part lines: the default policy
])
def test_large_vocabulary(N, K, H, V):
    g = torch.Generator(device="cuda").manual_seed(N)
    h = torch.randn(N, H, generator=g, device="cuda").bfloat16()
    w = (torch.randn(V, H, generator=g, device="cuda") / 64).bfloat16()
    print(f"N={N} K={K} H={H} V={V}", flush=True)
    out = osm.proj(h, w)
    cut = 24576
    parts = torch.cat([osm.proj(h, w[:cut]), osm.proj(h, w[cut:])], dim=1)
    assert torch.equal(out, parts)
    vals, idx = osm.proj_softmax_topk(h, w, K)
    v, i = osm.softmax_topk(out, K)
    assert torch.equal(idx, i)
    # both within the binary32 rule (RTOL) of the binary64 value
    assert torch.allclose(vals, v, rtol=2 * RTOL, atol=0)
