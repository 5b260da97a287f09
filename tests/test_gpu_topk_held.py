"""Rows and chunks held in registers (top-k of Alg. 4 and of the elements): at
the edges of every vectors-per-lane step, of the four- and eight-wavefront
shapes and of the streamed rows beyond them, aligned and not, against the
oracle: indices bit-exact, values within the binary32 rule."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_02867_amd as osm
from paper_1805_02867_amd import synth
from parity import assert_topk_equal, best_us, host_dtype, to_host

pytestmark = pytest.mark.gpu

STEPS = (1, 2, 3, 4, 6, 8, 12, 16)  # vectors per lane (13 too, by eight wavefronts)


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need an MI355X; none is visible")
    return torch.device("cuda:0")


def check(x, K, kernel, param, what):
    print(what, flush=True)
    vals, idx = osm.softmax_topk(x, K, kernel=kernel, param=param)
    torch.cuda.synchronize()
    v64, z64 = oracle.topk(to_host(x), K, host_dtype(x))
    assert_topk_equal(to_host(vals), to_host(idx), v64, z64, what)


def rows(N, V, dtype, dev, seed):
    """Ordinary rows, one on a coarse grid (ties across the K-th place), one of
    equal elements and one with a few finite elements among -inf."""
    x = synth.logits(N, V, sigma=2.0, seed=seed, dtype=dtype, device=dev)
    g = torch.Generator(device=dev).manual_seed(seed)
    x[1] = (torch.randint(-3, 4, (V,), generator=g, device=dev) * 0.5).to(x.dtype)
    x[2] = 0.75
    x[3] = float("-inf")
    x[3, ::max(1, V // 3)] = -2.0
    return x


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("lanes", [64, 256, 512])
def test_row_length_edges(dev, dtype, lanes):
    """lanes = 512: rows that eight wavefronts hold (forced as a workgroup per row)."""
    E = 4 if dtype == "f32" else 8
    for step in STEPS if lanes < 512 else (8, 9, 12, 13, 16):
        for d in (-1, 0, 1, E):
            V = lanes * step * E + d
            K = (1, 5, 64, 33)[(step + d) % 4]
            x = rows(5, V, dtype, dev, seed=V + K)
            check(x, K, osm.KERNEL_ROWS, min(lanes, 256), f"{dtype} lanes {lanes} V={V} K={K}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vectors", [1, 300, 4096, 4097, 6656, 6657, 8192, 8193])
def test_chunk_length_edges(dev, dtype, vectors):
    """Chunks of `vectors` 16-byte vectors, the last one short; 520 chunks at
    the smallest, so that the merge takes more keys than one wavefront holds."""
    E = 4 if dtype == "f32" else 8
    S = 520 if vectors < 100 else 3
    V = (S - 1) * vectors * E + 2 * E + 1
    for K in (1, 6, 64):
        x = rows(5, V, dtype, dev, seed=V + K)
        check(x, min(K, V), osm.KERNEL_SPLIT, S, f"{dtype} chunks of {vectors} V={V} K={K}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_plain_topk_skips_nan(dev, dtype):
    """topk_fwd: NaN is never selected; missing places hold -1 and NaN."""
    for V in (40, 1000, 20001):
        K = 20
        x = rows(6, V, dtype, dev, seed=V)
        x[4] = float("nan")
        x[4, 7:7 + 11] = torch.arange(11, device=dev).to(x.dtype)
        x[5, ::3] = float("nan")
        vals, idx = osm.topk(x, K)
        torch.cuda.synchronize()
        xh = x.float().cpu().numpy().astype(np.float64)
        for r in range(6):
            ok = np.flatnonzero(~np.isnan(xh[r]))
            z = ok[np.argsort(-xh[r][ok], kind="stable")][:K]
            got = to_host(idx)[r]
            assert got[:z.size].tolist() == z.tolist() and (got[z.size:] == -1).all(), (V, r)
            v = to_host(vals)[r]
            assert (v[:z.size] == xh[r][z]).all() and np.isnan(v[z.size:]).all(), (V, r)


@pytest.mark.parametrize("N,V,K", [(300, 50257, 5), (300, 50257, 9), (350, 65000, 8), (281, 49200, 8),
                                   (282, 49200, 8), (383, 49200, 5), (384, 49200, 5), (300, 40000, 5)])
def test_second_round_of_chunks(dev, N, V, K):
    """Two chunks a row, a little more of them than fit on the chip at once."""
    print(f"{N}x{V} K={K}", flush=True)
    x = synth.logits(N, V, sigma=2.0, seed=V, device=dev)
    vals, idx = osm.softmax_topk(x, K)
    torch.cuda.synchronize()
    pick = [0, 1, N // 2, N - 1]
    v64, z64 = oracle.topk(to_host(x[pick]), K, host_dtype(x))
    assert_topk_equal(to_host(vals)[pick], to_host(idx)[pick], v64, z64, f"{N}x{V} K={K}")


@pytest.mark.parametrize("K", [30, 64])
def test_thirteen_vectors_a_lane(dev, K):
    """Rows a little past 12 vectors a lane took 1.2 to 1.35 times the time of
    those with 12, since they loaded 16."""
    print(f"K={K}", flush=True)
    x = synth.logits(4000, 24576, sigma=2.0, seed=1, device=dev)
    twelve = best_us(lambda: osm.softmax_topk(x, K))
    x = synth.logits(4000, 25000, sigma=2.0, seed=1, device=dev)
    more = best_us(lambda: osm.softmax_topk(x, K))
    print(f"{twelve:.1f} us, {more:.1f} us", flush=True)
    assert more <= 1.14 * twelve
