"""fp32 calls with channels last that are lent work space: the tensors change their layout before and after the
convolution (a tiled transpose), or waves on their own store channels last themselves."""
import numpy as np
import pytest

import oracle
import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, make_input, make_layer

from gpu_util import assert_close, say, to_device

# (n, c_in, c_out, h, w, stride): remainders of the transpose's tiles of 64 on both sides, pixels that are no whole
# quads of channels, both strides; many images of few outputs and few images of many
SHAPES = [(1, 65, 63, 9, 7, 1), (2, 64, 64, 8, 8, 1), (3, 33, 17, 5, 13, 1), (2, 130, 20, 14, 14, 2), (1, 99, 70, 17, 31, 2),
          (9, 36, 12, 4, 4, 1), (1, 5, 9, 13, 6, 1), (2, 128, 128, 28, 28, 1), (8, 40, 200, 40, 36, 1), (4, 17, 130, 61, 59, 1)]


def make(shape, seed):
    n, ci, co, h, w, stride = shape
    spec = LayerSpec("ws", n, ci, co, h, w, stride=stride, keep_div=2.5, count_dist="bernoulli")
    return spec, make_layer(spec, seed), make_input(spec, seed)


def test_no_work_space_without_a_device():
    spec, L, _ = make(SHAPES[7], 1)
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32", host_only=True)
    assert P.lib().pconv_conv2d_workspace(h.ptr, 2, 28, 28, 1, P.NHWC, P.F32) == 0
    h.free()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_work_space_changes_the_layout_and_nothing_else(shape):
    import torch
    n, ci, co, hh, ww, stride = shape
    spec, L, x = make(shape, 7700 + ci)
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    b = torch.from_numpy(L["bias"]).cuda()
    xd = to_device(x, "f32")
    xl = xd.permute(0, 2, 3, 1).contiguous()
    size = P.lib().pconv_conv2d_workspace(h.ptr, n, hh, ww, stride, P.NHWC, P.F32)
    say(f"[case] work space {shape}: {size} bytes")
    assert size > 0
    assert P.lib().pconv_conv2d_workspace(h.ptr, n, hh, ww, stride, P.NCHW, P.F32) == 0
    for relu in (False, True):
        y = P.conv2d(h, xl, b, stride=stride, relu=relu, layout="nhwc")
        first = P.conv2d(h, xd, b, stride=stride, relu=relu)
        torch.cuda.synchronize()
        # the same kernels on the same numbers
        assert torch.equal(y.permute(0, 3, 1, 2), first)
        wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
        yr, sr = oracle.conv2d(x, wt, L["bias"], stride=stride, pad=1, relu=relu)
        assert_close(first.cpu().numpy().astype(np.float64), yr, sr, "f32", f"ws{shape}")
    # too little work space, or none: as pconv_conv2d
    want, got = torch.empty_like(y), torch.empty_like(y)
    st = torch.cuda.current_stream().cuda_stream
    P.pconv_conv2d(h, xl.data_ptr(), want.data_ptr(), b.data_ptr(), n, hh, ww, stride, 1, "nhwc", "f32", True, st)
    work = torch.full((size + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    for ptr, lent in ((None, size), (work.data_ptr(), size - 1)):
        got.fill_(float("nan"))
        assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), got.data_ptr(), b.data_ptr(), n, hh, ww, stride, 1, P.NHWC, P.F32, 1, st or None, ptr, lent) == P.OK
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    assert bool((work == 0xA5).all())
    # exactly as much as was asked for: nothing behind it is written
    assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), got.data_ptr(), b.data_ptr(), n, hh, ww, stride, 1, P.NHWC, P.F32, 1, st or None, work.data_ptr(), size) == P.OK
    torch.cuda.synchronize()
    assert torch.equal(got, y) and bool((work[size:] == 0xA5).all())
    # refused: work space off its alignment, and what pconv_conv2d refuses
    assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), got.data_ptr(), None, n, hh, ww, stride, 1, P.NHWC, P.F32, 0, st or None, work.data_ptr() + 8, size) == P.INVALID_ARG
    assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), xl.data_ptr(), None, n, hh, ww, stride, 1, P.NHWC, P.F32, 0, st or None, work.data_ptr(), size) == P.INVALID_ARG
    assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), got.data_ptr(), None, n, hh, ww, stride, 0, P.NHWC, P.F32, 0, st or None, work.data_ptr(), size) == P.INVALID_ARG
    h.free()


# (shape, waves, ks_log2, tiles cut rows, the convolution stores channels last itself): four slots and two (ks_log2 5),
# whole rows and cut ones, every shift of the last patch of a row, stride 2; and what changes its layout afterwards: few
# waves, an even width with stride 2, large outputs
FORMS = [((4, 33, 64, 32, 70, 1), 16, 4, 0, True), ((8, 128, 128, 28, 27, 2), 16, 4, 0, True), ((8, 128, 128, 28, 28, 1), 16, 4, 0, True),
         ((1, 40, 64, 83, 136, 1), 16, 4, 1, True), ((1, 99, 128, 67, 97, 1), 16, 4, 1, True), ((1, 99, 128, 67, 98, 1), 16, 4, 1, True),
         ((1, 99, 128, 67, 99, 1), 16, 4, 1, True), ((8, 128, 33, 37, 87, 2), 16, 4, 1, True), ((1, 99, 128, 52, 76, 1), 16, 5, 1, True),
         ((1, 64, 16, 10, 300, 1), 16, 5, 1, True), ((1, 64, 16, 10, 298, 1), 16, 5, 1, True), ((1, 64, 16, 10, 299, 2), 16, 5, 1, True),
         ((2, 64, 64, 8, 8, 1), 16, 5, 0, True), ((2, 130, 20, 14, 14, 2), 16, 5, 0, False), ((8, 128, 128, 28, 28, 2), 16, 4, 0, False),
         ((8, 128, 33, 37, 89, 2), 8, 4, 0, False), ((4, 17, 130, 61, 59, 1), 8, 4, 1, False), ((8, 40, 200, 40, 36, 1), 4, 4, 0, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,waves,ks_log2,cut,itself", FORMS)
def test_work_space_is_what_the_form_of_a_call_uses(shape, waves, ks_log2, cut, itself):
    import torch
    n, ci, co, hh, ww, stride = shape
    spec, L, x = make(shape, 7800 + ci)
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    plan = P.pconv_debug_plan(h, n, hh, ww, stride)
    assert (plan.waves, plan.ks_log2, plan.lone_cut) == (waves, ks_log2, cut)
    b = torch.from_numpy(L["bias"]).cuda()
    xd = to_device(x, "f32")
    xl = xd.permute(0, 2, 3, 1).contiguous()
    size = P.lib().pconv_conv2d_workspace(h.ptr, n, hh, ww, stride, P.NHWC, P.F32)
    first = P.conv2d(h, xd, b, stride=stride)
    assert size == -(-xd.numel() * 4 // 256) * 256 + (0 if itself else first.numel() * 4)
    say(f"[case] form {shape}: waves={waves} ks={ks_log2} cut={cut} stores channels last={itself}")
    work = torch.full((size + 1024,), 0xA5, dtype=torch.uint8, device="cuda")
    y = torch.full_like(first.permute(0, 2, 3, 1).contiguous(), float("nan"))
    assert P.lib().pconv_conv2d_ws(h.ptr, xl.data_ptr(), y.data_ptr(), b.data_ptr(), n, hh, ww, stride, 1, P.NHWC, P.F32, 0,
                                   torch.cuda.current_stream().cuda_stream or None, work.data_ptr(), size) == P.OK
    torch.cuda.synchronize()
    assert torch.equal(y.permute(0, 3, 1, 2), first) and bool((work[size:] == 0xA5).all())
    wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
    yr, sr = oracle.conv2d(x, wt, L["bias"], stride=stride, pad=1)
    assert_close(first.cpu().numpy().astype(np.float64), yr, sr, "f32", f"form{shape}")
    h.free()


# ((n, c_in, c_out, h, w, stride), keep, us as it is, us channels first): the layout stays
AS_IT_IS = [((44, 4, 5, 158, 126, 1), 3.6, 31, 59), ((4, 5, 13, 223, 178, 2), 8.0, 12, 19), ((42, 7, 35, 66, 79, 2), 3.6, 21, 30),
            ((13, 4, 35, 220, 176, 2), 3.6, 35, 48), ((25, 8, 18, 97, 99, 1), 2.5, 30, 35), ((39, 76, 13, 70, 70, 1), 2.5, 58, 69),
            ((7, 72, 8, 117, 117, 1), 2.5, 26, 31), ((33, 36, 7, 50, 50, 1), 2.5, 18, 21)]
# it changes
CHANNELS_FIRST = [((8, 128, 128, 28, 28, 1), 3.6, 34, 20), ((19, 5, 25, 209, 212, 1), 3.6, 151, 84), ((4, 4, 471, 223, 223, 1), 3.6, 680, 359),
                  ((16, 200, 50, 112, 112, 1), 3.6, 802, 210), ((5, 6, 12, 38, 38, 1), 3.6, 20, 11)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,keep,as_it_is,first", AS_IT_IS + CHANNELS_FIRST)
def test_the_layout_changes_where_that_is_faster(shape, keep, as_it_is, first):
    n, ci, co, hh, ww, stride = shape
    L = make_layer(LayerSpec("ws", 1, ci, co, 8, 8, stride=stride, keep_div=keep), 7700 + ci)
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    assert (P.lib().pconv_conv2d_workspace(h.ptr, n, hh, ww, stride, P.NHWC, P.F32) > 0) == (first < as_it_is)
    h.free()


@pytest.mark.gpu
def test_work_space_calls_under_capture():
    """The work space comes out of the graph's own pool; every replay sees its own input."""
    import torch
    shape = (2, 40, 200, 20, 24, 1)
    spec, L, x = make(shape, 7900)
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    b = torch.from_numpy(L["bias"]).cuda()
    xs = torch.zeros((2, 20, 24, 40), device="cuda")
    ys = torch.empty((2, 20, 24, 200), device="cuda")
    P.conv2d(h, xs, b, layout="nhwc", out=ys)
    torch.cuda.synchronize()
    say("[case] work space under capture")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        P.conv2d(h, xs, b, layout="nhwc", out=ys)
    for k in range(3):
        xk = torch.from_numpy(make_input(spec, 7901 + k)).cuda().permute(0, 2, 3, 1).contiguous()
        xs.copy_(xk); ys.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        got = ys.clone()
        assert torch.equal(got, P.conv2d(h, xk, b, layout="nhwc"))
    h.free()
