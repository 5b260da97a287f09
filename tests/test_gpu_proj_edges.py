"""The 256 x 256 projection core (calls of 512 tiles and more, and the fused
top-k past 128 rows) at the edges of its K steps and tiles, and the fused
epilogue on logits in rising and falling order, all equal and infinite.  Every product
and sum is exact in binary32 whatever its order, so logits must equal the
binary64 ones bit for bit and top-k indices the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_02867_amd as osm
from parity import rel_err_f32, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need an MI355X; none is visible")
    return torch.device("cuda:0")


def exact_inputs(N, H, V, seed, dev):
    """Small integers times powers of two: |logit| < 2^6, in steps of 2^-7."""
    g = torch.Generator(device=dev).manual_seed(seed)
    h = torch.randint(-4, 5, (N, H), generator=g, device=dev).to(torch.bfloat16) * 0.125
    w = torch.randint(-4, 5, (V, H), generator=g, device=dev).to(torch.bfloat16) * 0.0625
    return h, w


def logits64(h, w):
    return torch.matmul(h.double(), w.double().t())


def check_topk(h, w, K, what):
    print(what, flush=True)
    vals, idx = osm.proj_softmax_topk(h, w, K)
    torch.cuda.synchronize()
    v64, z64 = oracle.topk(to_host(logits64(h, w)), K, "f64")
    assert np.array_equal(to_host(idx), z64), what
    assert (rel_err_f32(to_host(vals), v64) <= 1).all(), what


@pytest.mark.parametrize("H", [8, 64, 72, 128, 136, 192, 1032])
def test_logits_k_step_edges(dev, H):
    N, V = 4097, 8001  # 17 x 32 tiles, one row and 65 columns into the last
    h, w = exact_inputs(N, H, V, seed=H, dev=dev)
    out = torch.full((N, V), 7.0, device=dev)
    print(f"logits H={H}", flush=True)
    osm.proj(h, w, out)
    torch.cuda.synchronize()
    assert torch.equal(out.double(), logits64(h, w))


@pytest.mark.parametrize("H", [8, 64, 136, 256])
@pytest.mark.parametrize("K", [1, 5, 8, 9, 16])
def test_topk_tile_edges(dev, H, K):
    for N, V in ((129, 257), (256, 2560), (257, 5121), (513, 33), (1025, 700)):
        check_topk(*exact_inputs(N, H, V, seed=N + V + H + K, dev=dev), min(K, V),
                   f"fused N={N} H={H} V={V} K={K}")


@pytest.mark.parametrize("N", [40, 100, 200, 1100])
@pytest.mark.parametrize("K", [1, 5, 8, 16])
def test_topk_of_ordered_logits(dev, N, K):
    """Rising logits make every entry a new maximum, equal ones are all ties."""
    V, H = 9000, 64
    h = torch.zeros((N, H), dtype=torch.bfloat16, device=dev)
    h[:, 0], h[:, 1] = 1.0, 1.0 / 128
    v = torch.arange(V, device=dev)
    for what, order in (("rising", v), ("falling", V - 1 - v), ("equal", v * 0)):
        w = torch.zeros((V, H), dtype=torch.bfloat16, device=dev)
        w[:, 0] = torch.div(order, 128, rounding_mode="floor").to(torch.bfloat16)
        w[:, 1] = (order % 128).to(torch.bfloat16)
        check_topk(h, w, K, f"{what} N={N} K={K}")


@pytest.mark.parametrize("K", [1, 8, 9, 16])
@pytest.mark.parametrize("V", [17, 63, 64, 65, 16384, 16385, 32769, 40960, 40961, 98304, 98305])
def test_small_batch_tile_heights(dev, V, K):
    """Batches of up to 64 rows: on both sides of each line between the tile
    heights of 64, 128 and 256, with a row or a remainder in the last tile."""
    for N, H in ((1, 72), (64, 1032)):
        check_topk(*exact_inputs(N, H, V, seed=N + V + H + K, dev=dev), min(K, V),
                   f"fused N={N} H={H} V={V} K={K}")


@pytest.mark.parametrize("K", [9, 12, 16])
@pytest.mark.parametrize("N,H,V", [
    (257, 2048, 33000), (1100, 2056, 16001),   # a tile a workgroup, ragged both ways
    (600, 2048, 30001),                        # two tiles a workgroup
    (256, 2048, 65537), (256, 2048, 65536),    # one strip: on both sides of the layout's line
    (1100, 2040, 16001)])                      # H below it
def test_lists_of_16_on_the_two_group_core(dev, N, H, V, K):
    check_topk(*exact_inputs(N, H, V, seed=N + V + K, dev=dev), K, f"fused N={N} H={H} V={V} K={K}")


@pytest.mark.parametrize("N,H,V,K", [
    (40, 64, 9000, 1), (40, 64, 9000, 8), (40, 64, 9000, 16),          # tiles of 64 and 256
    (40, 72, 45000, 5), (100, 64, 9000, 5), (100, 64, 9000, 16),       # of 128; 128 rows a strip
    (200, 64, 9000, 1), (200, 64, 9000, 8), (1100, 64, 9000, 16), (257, 2048, 33000, 12)])
def test_infinite_logits(dev, N, H, V, K):
    """-infinity is passed over and adds nothing; +infinity comes first, in index
    order, and makes every probability of its row NaN, as inf - inf is."""
    h, w = exact_inputs(N, H, V, seed=N + V + K, dev=dev)
    h[:, 0] = 0.5
    v = torch.arange(V, device=dev)
    w[(v < 700) | (v % 3 == 0) | (v > V - 70), 0] = float("-inf")
    print(f"-inf N={N} H={H} V={V} K={K}", flush=True)
    vals, idx = osm.proj_softmax_topk(h, w, K)
    torch.cuda.synchronize()
    x = to_host(logits64(h, w))
    v64, z64 = oracle.topk(x, K, "f64")
    assert np.array_equal(to_host(idx), z64)
    assert (rel_err_f32(to_host(vals), v64) <= 1).all()

    w[[701, 702, V // 2, V - 71], 0] = float("inf")
    w[1000:1040:2, 0] = float("inf")                   # more than K of them in a lane or two
    print(f"+inf N={N} H={H} V={V} K={K}", flush=True)
    vals, idx = osm.proj_softmax_topk(h, w, K)
    torch.cuda.synchronize()
    x = to_host(logits64(h, w))
    z = np.argsort(-x, axis=1, kind="stable")[:, :K]
    assert np.array_equal(to_host(idx), z)
    assert np.isnan(to_host(vals)).all()
