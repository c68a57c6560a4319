"""A row's result does not depend on how many rows are in the call: small calls take another kernel than large ones
(latency against throughput), and the two form every result from the same int32 group sums, folded in the same order,
so a sample alone and the same sample in a large batch are equal bit for bit."""
import numpy as np
import pytest

import dgq_inputs as di
from support import CLASSES, CONV, GATED, PLAIN, REQUANT, kernel_of

pytestmark = pytest.mark.gpu

FEW, MANY = 70, 8192


@pytest.fixture(scope="module")
def dgq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2501_04304_amd as m
    m.lib()
    return m


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _same_bits(few, many):
    import torch
    assert torch.equal(few.view(torch.int32), many[:few.shape[0]].view(torch.int32))


def _two_kernels(g, few, many, out_channels, kind):
    a, b = (kernel_of(r, out_channels, g.info.k_padded, g.info.n_groups, kind) for r in (few, many))
    assert a < 10 <= b


def _calibrate(dgq, x, kind, ab):
    if kind == "channel":
        return dgq.dgq_calibrate_kmeans(x, ab, 16, dgq.DIM_CHANNEL)
    if kind == "pixel":
        return dgq.dgq_calibrate_kmeans(x, ab, 16, dgq.DIM_PIXEL)
    return dgq.dgq_calibrate_groups(x, ab, kind, 2)


@pytest.mark.parametrize("ab", [8, 4])
@pytest.mark.parametrize("kind,C", [
    (64, 320),          # every chunk a group
    (128, 768),         # groups of two chunks and a shorter one
    (256, 1288),        # groups of four chunks
    ("channel", 1280),  # groups of any length
    ("pixel", 1280),    # one group, sixteen classes
    (128, 64), (128, 200),  # about as many chunks as are read ahead
])
def test_linear(dgq, kind, C, ab):
    import torch
    run = di.linear_case(40 + C, 2, MANY // 2, C, 1280)
    x = _dev(run["X"])
    g = _calibrate(dgq, x, kind, ab)
    _two_kernels(g, FEW, MANY, 1280, CLASSES if kind == "pixel" else PLAIN)
    bias = _dev(np.random.default_rng(C).standard_normal(1280).astype(np.float32))
    w = dgq.dgq_pack_weight(g, _dev(run["W"]), bias, 8)
    few = dgq.dgq_linear(g, w, *dgq.dgq_quantize_act(g, x[:FEW]))
    many = dgq.dgq_linear(g, w, *dgq.dgq_quantize_act(g, x))
    _same_bits(few, many)
    if kind != "pixel":
        # every group's int32 sum is what went into the result
        dump = torch.full((FEW, 1280, g.info.n_groups), -7, dtype=torch.int32, device="cuda")
        codes, cls = dgq.dgq_quantize_act(g, x[:FEW])
        y = dgq.dgq_linear(g, w, codes, cls, acc_dump=dump)
        assert torch.equal(y.view(torch.int32), few.view(torch.int32))
        dump_many = torch.full((MANY, 1280, g.info.n_groups), -7, dtype=torch.int32, device="cuda")
        dgq.dgq_linear(g, w, *dgq.dgq_quantize_act(g, x), acc_dump=dump_many)
        assert torch.equal(dump, dump_many[:FEW])
    w.free()
    g.free()


@pytest.mark.parametrize("ab", [8, 4])
@pytest.mark.parametrize("kind,C", [(64, 320), (128, 768), ("channel", 640)])
def test_gated(dgq, kind, C, ab):
    import torch
    run = di.linear_case(50 + C, 2, MANY // 2, C, 2560)
    x = _dev(run["X"])
    g = _calibrate(dgq, x, kind, ab)
    _two_kernels(g, FEW, MANY, 2560, GATED)
    w = dgq.dgq_pack_weight(g, _dev(run["W"]), None, 8)
    few = dgq.dgq_linear_geglu(g, w, *dgq.dgq_quantize_act(g, x[:FEW]))
    many = dgq.dgq_linear_geglu(g, w, *dgq.dgq_quantize_act(g, x))
    _same_bits(few, many)
    g2 = dgq.dgq_calibrate_groups(many[:2048].contiguous(), ab, 128, 1)
    _two_kernels(g, FEW, MANY, 2 * g2.info.k_padded, REQUANT)
    w2 = dgq.dgq_pack_weight_gated_for(g, g2, _dev(run["W"]), None, 8)
    codes_few, _ = dgq.dgq_linear_geglu_requant(g, w2, *dgq.dgq_quantize_act(g, x[:FEW]), g2)
    codes_many, _ = dgq.dgq_linear_geglu_requant(g, w2, *dgq.dgq_quantize_act(g, x), g2)
    whole = FEW // (16 if ab == 8 else 32)  # row blocks with no row past the end
    assert torch.equal(codes_few[:whole], codes_many[:whole])
    for h in (w, w2, g, g2):
        h.free()


@pytest.mark.parametrize("ab", [8, 4])
@pytest.mark.parametrize("kind,C", [("blocks", 128), ("blocks", 320), ("channel", 64)])
def test_convolution(dgq, kind, C, ab):
    B, H, W, O = 32, 8, 32, 640
    run = di.linear_case(60 + C, B, H * W, C, 8)
    x = _dev(run["X"])
    g = dgq.dgq_calibrate_kmeans(x, ab, 8, dgq.DIM_CHANNEL) if kind == "channel" else dgq.dgq_calibrate_groups(x, ab, 64, 1)
    g9 = dgq.dgq_groups_for_conv3x3(g)
    _two_kernels(g9, H * W, B * H * W, O, CONV)
    k = np.random.default_rng(C).standard_normal((O, 9 * C)).astype(np.float32) * np.float32(0.02)
    w = dgq.dgq_pack_weight(g9, _dev(k), None, 8)
    out = []
    for b in (1, B):
        codes3, cls = dgq.dgq_quantize_act_conv3x3(g, g9, x[:b * H * W], b, H, W)
        out.append(dgq.dgq_linear_conv3x3(g9, w, codes3, cls, b, H, W))
        codes, cls = dgq.dgq_quantize_act(g, x[:b * H * W])
        unfolded = dgq.dgq_linear(g9, w, dgq.dgq_conv3x3_codes(g9, codes, b, H, W), cls)
        _same_bits(unfolded, out[-1])
    _same_bits(*out)
    for h in (w, g9, g):
        h.free()
