"""The softmax plan's line between a workgroup per row and split rows, on both
of its sides: the plan says which kernel runs, and its output matches the
binary64 oracle, on rows with a heavy tail, an equal row and mostly -inf."""
import pytest
import torch

import oracle
import paper_1805_02867_amd as osm
from paper_1805_02867_amd import synth
from parity import assert_softmax_close, best_us, host_dtype, to_host

pytestmark = pytest.mark.gpu

R, S = osm.KERNEL_ROWS, osm.KERNEL_SPLIT


@pytest.mark.parametrize("N,V,dtype,kernel", [
    (2, 16384, "f32", R), (2, 20480, "bf16", R), (2, 20481, "f32", S), (95, 20481, "bf16", S),
    (96, 20481, "f32", R), (96, 57344, "f32", R), (96, 57345, "f32", S), (127, 50000, "f32", R),
    (128, 49152, "f32", R), (128, 49153, "f32", S), (160, 65536, "f32", S), (160, 65537, "f32", R),
    (161, 57345, "f32", R),
    (256, 131071, "f32", R), (257, 57345, "f32", S), (128, 131073, "f32", S),
    (96, 24576, "bf16", R), (96, 24577, "bf16", S), (128, 24577, "bf16", R), (191, 57345, "bf16", S),
    (192, 57345, "bf16", R), (300, 24577, "bf16", S), (410, 24577, "bf16", R), (511, 16385, "bf16", R),
])
def test_plan_line(N, V, dtype, kernel):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the batch sizes stand for 256 CUs")
    x = synth.logits(N, V, sigma=3.0, seed=V + N, dtype=dtype, device="cuda")
    x[0, 1:] = float("-inf")
    x[1] = 0.5
    for mode in ("naive", "safe", "online"):
        print(f"{N}x{V} {dtype} {mode}", flush=True)
        assert osm.plan(N, V, dtype=x.dtype, mode=mode)[0] == kernel
        y = osm.softmax_fwd(x, mode=mode)
        pick = [0, 1, N // 2, N - 1]
        assert_softmax_close(to_host(y[pick]), oracle.softmax(to_host(x[pick]), host_dtype(x)),
                             f"{N}x{V} {dtype} {mode}")


@pytest.mark.parametrize("N,V,dtype,lanes", [
    (512, 768, "bf16", 32), (512, 769, "bf16", 128), (513, 1024, "bf16", 32), (3, 512, "f32", 32),
    (256, 640, "f32", 64), (256, 641, "f32", 256), (257, 800, "f32", 64), (512, 801, "f32", 256),
    (513, 2048, "f32", 64), (512, 4096, "f32", 256), (513, 2049, "f32", 128),
    (1024, 4093, "f32", 128), (1025, 4096, "f32", 64), (2, 1281, "bf16", 256),
    (1024, 8192, "bf16", 128), (2047, 4097, "bf16", 64), (2048, 4097, "bf16", 128),
    (2048, 6144, "bf16", 128), (2048, 6145, "bf16", 64),
])
def test_lanes_line(N, V, dtype, lanes):
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the batch sizes stand for 256 CUs")
    x = synth.logits(N, V, sigma=3.0, seed=V + N, dtype=dtype, device="cuda")
    x[0, 1:] = float("-inf")
    x[1] = 0.5
    for mode in ("naive", "safe", "online"):
        print(f"{N}x{V} {dtype} {mode}", flush=True)
        assert osm.plan(N, V, dtype=x.dtype, mode=mode) == (R, lanes)
        y = osm.softmax_fwd(x, mode=mode)
        pick = [0, 1, N // 2, N - 1]
        assert_softmax_close(to_host(y[pick]), oracle.softmax(to_host(x[pick]), host_dtype(x)),
                             f"{N}x{V} {dtype} {mode}")


def offset_pair(N, V, dtype):
    """x and a y that is not congruent with it modulo 16 bytes."""
    x = synth.logits(N, V, sigma=3.0, seed=V, dtype=dtype, device="cuda")
    y = torch.empty(N * V + 8, dtype=x.dtype, device="cuda")[3:3 + N * V].view(N, V)
    return x, y


@pytest.mark.parametrize("N,V,dtype", [
    (2, 16383, "bf16"), (2, 16384, "bf16"), (64, 16385, "f32"), (192, 32000, "bf16"),
    (255, 24580, "f32"), (256, 24580, "f32"), (300, 24577, "f32"), (410, 49160, "bf16")])
def test_incongruent_outputs(N, V, dtype):
    x, y = offset_pair(N, V, dtype)
    for mode in ("naive", "safe", "online"):
        print(f"{N}x{V} {dtype} {mode}", flush=True)
        osm.softmax_fwd(x, y, mode=mode)
        pick = [0, 1, N // 2, N - 1]
        assert_softmax_close(to_host(y[pick]), oracle.softmax(to_host(x[pick]), host_dtype(x)),
                             f"{N}x{V} {dtype} {mode}")


@pytest.mark.parametrize("N,V,S", [(128, 50000, 8), (144, 50000, 8), (128, 57344, 8)])
def test_half_the_chip_busy(N, V, S):
    """A workgroup per row took up to 1.3 times the time of split rows here."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the batch sizes stand for 256 CUs")
    x = synth.logits(N, V, sigma=3.0, seed=V, device="cuda")
    y = torch.empty_like(x)
    print(f"{N}x{V}", flush=True)
    auto = best_us(lambda: osm.softmax_fwd(x, y))
    split = best_us(lambda: osm.softmax_fwd(x, y, kernel=osm.KERNEL_SPLIT, param=S))
    print(f"{auto:.1f} us, split {split:.1f} us", flush=True)
    assert osm.plan(N, V)[0] == osm.KERNEL_SPLIT and auto <= 1.15 * split


@pytest.mark.parametrize("N,V,dtype,S", [(64, 16384, "bf16", 4), (192, 32000, "bf16", 6),
                                         (96, 57344, "f32", 11)])
def test_incongruent_outputs_keep_the_split(N, V, dtype, S):
    """A workgroup per row took about twice the time of split rows here."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the batch sizes stand for 256 CUs")
    x, y = offset_pair(N, V, dtype)
    print(f"{N}x{V} {dtype}", flush=True)
    auto = best_us(lambda: osm.softmax_fwd(x, y))
    split = best_us(lambda: osm.softmax_fwd(x, y, kernel=osm.KERNEL_SPLIT, param=S))
    print(f"{auto:.1f} us, split {split:.1f} us", flush=True)
    assert auto <= 1.3 * split
