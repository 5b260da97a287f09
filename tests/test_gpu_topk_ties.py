"""Top-k of rows in which many elements share one value (rows of one value,
coarse grids, masks): the lowest indices win, as the oracle has it, whichever
wavefront, vector or scalar end of the row they lie in; and of rows whose
largest elements lie side by side.  Both take little longer than other rows."""
import pytest
import torch

import oracle
import paper_1805_02867_amd as osm
from paper_1805_02867_amd import synth
from parity import assert_topk_equal, best_us, host_dtype, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need an MI355X; none is visible")
    return torch.device("cuda:0")


def tied_rows(V, dtype, dev, seed):
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=dev).manual_seed(seed)

    def pick(levels):
        return torch.randint(0, levels, (V,), generator=g, device=dev)
    x = torch.empty((10, V), dtype=t, device=dev)
    x[0] = -1.5                                          # one value
    x[1] = (pick(2) * 2 - 1) * 0.0                       # +0 and -0, which are equal
    x[2] = pick(7) * 0.5 - 2
    x[3] = pick(100) * 0.125
    x[4] = float("-inf")                                 # all but three masked
    x[4, [0, V // 2, V - 1]] = torch.tensor([1.0, 3.0, 2.0], dtype=t, device=dev)
    x[5] = torch.where(pick(50) == 0, pick(3), -9.0)     # a few values above many ties
    x[6] = -9.0                                          # larger ones at the row's end only
    x[6, -min(V, 40):] = torch.arange(min(V, 40), device=dev).to(t)
    x[7] = pick(7) * 0.5 - 2
    x[7, :V // 2] = -8.0                                 # ties in the second half
    x[8] = torch.finfo(t).min / 4                        # a finite mask, and half of the row
    x[8, ::2] = 0.25
    x[9] = pick(30) * 0.25
    return x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [1, 5, 50, 64])
@pytest.mark.parametrize("lanes,kernel,param", [
    (64, osm.KERNEL_ROWS, 64), (256, osm.KERNEL_ROWS, 256), (512, osm.KERNEL_ROWS, 256),
    (256, osm.KERNEL_SPLIT, 3), (512, osm.KERNEL_SPLIT, 3)])
def test_ties(dev, dtype, K, lanes, kernel, param):
    E = 4 if dtype == "f32" else 8
    chunks = param if kernel == osm.KERNEL_SPLIT else 1
    for step in (1, 2, 3, 7, 12, 16) if lanes < 512 else (9, 12, 13, 16):
        V = chunks * lanes * step * E - 3
        x = tied_rows(V, dtype, dev, seed=V + K)
        what = f"{dtype} K={K} lanes {lanes} V={V} kernel {kernel}"
        print(what, flush=True)
        vals, idx = osm.softmax_topk(x, K, kernel=kernel, param=param)
        torch.cuda.synchronize()
        v64, z64 = oracle.topk(to_host(x), K, host_dtype(x))
        assert_topk_equal(to_host(vals), to_host(idx), v64, z64, what)


@pytest.mark.parametrize("N,V,dtype,K", [
    (4000, 32000, "f32", 5), (4000, 32000, "f32", 50), (4000, 10000, "f32", 5),
    (4000, 4000, "f32", 1), (64, 128256, "f32", 5), (4000, 32000, "bf16", 5)])
def test_ties_cost_little(dev, N, V, dtype, K):
    """Rows of one value against ordinary rows: looked at element by element,
    they took 1.7 to 3.4 times as long."""
    x = synth.logits(N, V, sigma=2.0, seed=1, dtype=dtype, device=dev)
    print(f"{N}x{V} {dtype} K={K}", flush=True)
    plain = best_us(lambda: osm.softmax_topk(x, K))
    x.fill_(0.5)
    tied = best_us(lambda: osm.softmax_topk(x, K))
    print(f"{plain:.1f} us, ties {tied:.1f} us", flush=True)
    assert tied <= 1.5 * plain


@pytest.mark.parametrize("N,V,dtype,levels", [(4000, 4000, "f32", 7), (2000, 60000, "bf16", 100)])
def test_sparser_ties_cost_little(dev, N, V, dtype, levels):
    """One element in 7, and in 100, equal to the largest: the first vectors of a
    team hold fewer than 50, the next few do (1.9 times as long without them)."""
    x = synth.logits(N, V, sigma=2.0, seed=1, dtype=dtype, device=dev)
    print(f"{N}x{V} {dtype} {levels} levels", flush=True)
    plain = best_us(lambda: osm.softmax_topk(x, 50))
    g = torch.Generator(device=dev).manual_seed(V)
    x.copy_(torch.randint(0, levels, (N, V), generator=g, device=dev) * 0.0625)
    tied = best_us(lambda: osm.softmax_topk(x, 50))
    print(f"{plain:.1f} us, ties {tied:.1f} us", flush=True)
    assert tied <= 1.45 * plain


def falling(N, V, dtype, dev):
    """Logits that fall with the index, as of a vocabulary in order of frequency."""
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device=dev).manual_seed(V)
    x = torch.randn((N, V), generator=g, device=dev)
    return (x - 1.2 * torch.log1p(torch.arange(V, device=dev))).to(t)


@pytest.mark.parametrize("V,dtype", [(1000, "f32"), (4100, "f32"), (32000, "f32"), (128256, "f32"),
                                     (1000, "bf16"), (9000, "bf16"), (60000, "bf16")])
def test_largest_elements_side_by_side(dev, V, dtype):
    x = torch.cat([falling(6, V, dtype, dev), falling(6, V, dtype, dev).flip(1),
                   torch.arange(V, device=dev).to(torch.float32).mul(-8.0 / V)[None].to(
                       torch.float32 if dtype == "f32" else torch.bfloat16)])
    for K in (1, 20, 50, 64):
        print(f"{V} {dtype} K={K}", flush=True)
        vals, idx = osm.softmax_topk(x, K)
        torch.cuda.synchronize()
        v64, z64 = oracle.topk(to_host(x), K, host_dtype(x))
        assert_topk_equal(to_host(vals), to_host(idx), v64, z64, f"{V} {dtype} K={K}")


@pytest.mark.parametrize("N,V,dtype", [(4000, 1000, "f32"), (2000, 60000, "bf16")])
def test_largest_side_by_side_cost_little(dev, N, V, dtype):
    """Against ordinary rows: 1.45 times as long with every list sorted in full."""
    print(f"{N}x{V} {dtype}", flush=True)
    x = synth.logits(N, V, sigma=2.0, seed=1, dtype=dtype, device=dev)
    plain = best_us(lambda: osm.softmax_topk(x, 50))
    x = falling(N, V, dtype, dev)
    side = best_us(lambda: osm.softmax_topk(x, 50))
    print(f"{plain:.1f} us, side by side {side:.1f} us", flush=True)
    assert side <= 1.4 * plain
