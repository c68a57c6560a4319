"""Tensors that are too small for the call are refused on the host: the C ABI sees no sizes, a kernel would read or
write past their end."""
import numpy as np
import pytest

import dgq_inputs as di

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dgq():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2501_04304_amd as m
    m.lib()
    return m


def _f(*shape):
    import torch
    return torch.ones(shape, dtype=torch.float32, device="cuda")


B, N, H, D, NK = 2, 40, 3, 16, 9


@pytest.mark.parametrize("short", ["out", "scale_out"])
def test_xattn(dgq, short):
    q, k, v = _f(B, N, H, D), _f(B, NK, H, D), _f(B, NK, H, D)
    bad = dict(out=_f(B, N, H, D - 1), scale_out=_f(B - 1))[short]
    with pytest.raises(ValueError, match=short):
        dgq.dgq_xattn_logq(q, k, v, None, 8, **{short: bad})


@pytest.mark.parametrize("short", ["key_bias", "scale_in", "out", "scale_out", "codes_dump"])
def test_xattn_static(dgq, short):
    import torch
    q, k, v = _f(B, N, H, D), _f(B, NK, H, D), _f(B, NK, H, D)
    args = dict(key_bias=_f(NK), scale_in=_f(B))
    args[short] = dict(key_bias=_f(NK - 1), scale_in=_f(B - 1), out=_f(B, N - 1, H, D), scale_out=_f(B - 1),
                       codes_dump=torch.zeros(B * H * N * (NK - 1) - 1, dtype=torch.uint8, device="cuda"))[short]
    with pytest.raises(ValueError, match=short):
        dgq.dgq_xattn_logq_static(q, k, v, args.pop("key_bias"), 8, args.pop("scale_in"), **args)


@pytest.mark.parametrize("short", ["out", "scale_out"])
def test_selfattn(dgq, short):
    q = _f(B, N, H, D)
    bad = dict(out=_f(B, N, H, D - 1), scale_out=_f(B - 1))[short]
    with pytest.raises(ValueError, match=short):
        dgq.dgq_selfattn_logq(q, q, q, 8, _f(B), **{short: bad})


@pytest.mark.parametrize("short", ["key_bias", "out", "scale_out"])
def test_xattn_intv(dgq, short):
    import torch
    q, k = _f(B, N, H, D), _f(B, NK, H, D)
    codes = torch.zeros((B, NK, H, D), dtype=torch.uint8, device="cuda")
    args = dict(key_bias=_f(NK))
    args[short] = dict(key_bias=_f(NK - 1), out=_f(B, N, H, D - 1), scale_out=_f(B - 1))[short]
    with pytest.raises(ValueError, match=short):
        dgq.dgq_xattn_logq_intv(q, k, codes, _f(B, H, 2), args.pop("key_bias"), **args)


def test_quantize_value(dgq):
    with pytest.raises(ValueError, match="v_hat"):
        dgq.dgq_quantize_value(_f(B, NK, H, D), v_hat=_f(B, NK, H, D - 1))


@pytest.mark.parametrize("short", ["codes3", "row_class"])
def test_convolution(dgq, short):
    import torch
    b, h, w, c, o = 1, 4, 32, 64, 8
    x = torch.from_numpy(np.ascontiguousarray(di.linear_case(5, b, h * w, c, 8)["X"])).cuda()
    g = dgq.dgq_calibrate_groups(x, 8, 64, 1)
    g9 = dgq.dgq_groups_for_conv3x3(g)
    wt = dgq.dgq_pack_weight(g9, _f(o, 9 * c), None, 8)
    args = list(dgq.dgq_quantize_act_conv3x3(g, g9, x, b, h, w))
    i = ["codes3", "row_class"].index(short)
    args[i] = args[i][:-1].contiguous()
    with pytest.raises(ValueError, match=short):
        dgq.dgq_linear_conv3x3(g9, wt, *args, b, h, w)
    for handle in (wt, g9, g):
        handle.free()
