"""The GPU tests that mean to reach a certain kernel of the contraction still do (on the CPU: the library's own choice
for their shapes, with the groups that the oracle's calibration gives), and between them they reach every one."""
import pytest

import dgq_inputs as di
import test_gpu_conv
import test_gpu_geglu
import test_gpu_kmeans
import test_gpu_linear
import test_gpu_requant
from support import CLASSES, CONV, GATED, PLAIN, REQUANT, kernel_of

DIRECT, RING = {0, 1, 2}, {10, 11, 12, 13}
SPLIT = {0, 2, 12, 13}  # the gated forms: two column blocks per wavefront


@pytest.mark.parametrize("ab", [8, 4])
def test_linear(oracle, ab):
    for B, N, C, O, G, kernel in test_gpu_linear.RAGGED:
        g = oracle.calibrate(di.linear_case(300 + C + O, B, N, C, O, calib=True)["X"], ab, G, 2)
        assert kernel_of(B * N, O, g.Kp, g.NG, PLAIN) == kernel, (B, N, C, O)
    assert {s[-1] for s in test_gpu_linear.RAGGED} == DIRECT | RING


def test_pixel_classes():
    for B, N, C, O, K, kernel in test_gpu_kmeans.RAGGED:
        assert kernel_of(B * N, O, (C + 63) // 64 * 64, 1, CLASSES) == kernel, (B, N, C, O)
    assert {s[-1] for s in test_gpu_kmeans.RAGGED} == DIRECT | RING


@pytest.mark.parametrize("ab", [8, 4])
def test_gated(oracle, ab):
    for B, N, C, O, G, kernel in test_gpu_geglu.RAGGED:
        g = oracle.calibrate(di.linear_case(700 + C + O, B, N, C, O, calib=True)["X"], ab, G, 2)
        assert kernel_of(B * N, O, g.Kp, g.NG, GATED) == kernel, (B, N, C, O)
    assert {s[-1] for s in test_gpu_geglu.RAGGED} == SPLIT


@pytest.mark.parametrize("bits,shapes,seed", [(8, test_gpu_requant.RAGGED, 900), (4, test_gpu_requant.RAGGED_TO_4_BIT, 950)])
def test_requantized(oracle, bits, shapes, seed):
    for B, N, C1, C2, G, ab, kind, kernel in shapes:
        _, _, _, g, _, g2 = test_gpu_requant.layers(oracle, B, N, C1, C2, G, ab, seed + C1 + C2, kind, next_bits=bits)
        assert kernel_of(B * N, 2 * g2.Kp, g.Kp, g.NG, REQUANT) == kernel, (B, N, C1, C2, kind)
    assert {s[-1] for s in shapes} == SPLIT


@pytest.mark.parametrize("ab", [8, 4])
def test_gathered_convolution(oracle, ab):
    for B, H, W, C, O, kind, kernel in test_gpu_conv.GATHERED:
        cal = di.linear_case(78, B, H * W, C, 8, calib=True)["X"]
        g = oracle.calibrate_kmeans(cal, ab, 1, 0) if kind == "one" else oracle.calibrate(cal, ab, 64, 1)
        assert kernel_of(B * H * W, O, 9 * g.Kp, 9 * g.NG, CONV) == kernel, (B, H, W, C, O)
    assert {s[-1] for s in test_gpu_conv.GATHERED} == DIRECT | RING
