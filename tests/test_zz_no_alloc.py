"""pconv_conv2d_static (the entry point for callers that cannot let the library allocate: its
hand-over words live in a static device array of the code object) against pconv_conv2d, through
the C ABI: same kernels, same order of additions, so the outputs must agree bit for bit - and
with the oracle within the fp32 bar.  Two calls in a row, the second on a smaller input.  And both entry
points under graph capture, where a call's arguments stay the same from replay to replay."""
import numpy as np
import pytest

import oracle
import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, base_seed, config_layers, make_input, make_layer

from gpu_util import assert_close, say, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _reset_tiling():
    yield
    P.pconv_debug_set_tiling(0, -1, -1)


@pytest.mark.parametrize("split_units", [1, 2])
def test_static_scratch_entry_point_two_calls_second_smaller(split_units):
    import torch
    spec = config_layers(2)[0]                       # 256 -> 256 at 56x56, batch 1
    P.pconv_debug_set_tiling(0, -1, split_units)     # workgroups share units: the hand-over words are used
    L = make_layer(spec, base_seed(2))
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    b = torch.from_numpy(L["bias"]).cuda()
    wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
    stream = torch.cuda.current_stream().cuda_stream
    for k, (hh, ww) in enumerate([(56, 56), (28, 20)]):
        x = make_input(LayerSpec("s", 1, 256, 256, hh, ww), base_seed(2) + k)
        xd = to_device(x, "f32")
        say(f"[case] pconv_conv2d_static call {k}: x={x.shape} split={split_units}")
        assert P.pconv_debug_plan(h, 1, hh, ww).split_units == split_units
        ref = P.conv2d(h, xd, b, relu=True)
        y = torch.full_like(ref, float("nan"))
        P.pconv_conv2d_static(h, xd.data_ptr(), y.data_ptr(), b.data_ptr(), 1, hh, ww, 1, 1, P.NCHW, P.F32,
                              True, stream)
        torch.cuda.synchronize()
        assert torch.equal(y, ref), f"call {k}: static-scratch result differs from pconv_conv2d"
        yr, sr = oracle.conv2d(x, wt, L["bias"], relu=True)
        assert_close(y.cpu().numpy().astype(np.float64), yr, sr, "f32", f"static call {k}")
    P.pconv_get_async_error(h)
    h.free()


@pytest.mark.parametrize("split_units", [1, 2])
@pytest.mark.parametrize("static", [False, True])
def test_replays_of_a_captured_call_see_their_own_input(static, split_units):
    """A layer whose workgroups share units: the hand-over words of one replay must not serve the next."""
    import torch
    spec = config_layers(2)[0]
    P.pconv_debug_set_tiling(0, -1, split_units)
    L = make_layer(spec, base_seed(2))
    h = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    assert P.pconv_debug_plan(h, 1, spec.h, spec.w).split_units == split_units
    b = torch.from_numpy(L["bias"]).cuda()
    wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
    x = torch.zeros((1, spec.c_in, spec.h, spec.w), device="cuda")
    y = torch.empty((1, spec.c_out, spec.h, spec.w), device="cuda")

    def call():
        f = P.pconv_conv2d_static if static else P.pconv_conv2d
        f(h, x.data_ptr(), y.data_ptr(), b.data_ptr(), 1, spec.h, spec.w, 1, 1, P.NCHW, P.F32, True,
          torch.cuda.current_stream().cuda_stream)
    call()
    torch.cuda.synchronize()
    say(f"[case] capture static={static} split={split_units}")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for k in range(3):
        xk = make_input(spec, base_seed(2) + 30 + k)
        x.copy_(torch.from_numpy(xk)); y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        yr, sr = oracle.conv2d(xk, wt, L["bias"], relu=True)
        assert_close(y.cpu().numpy().astype(np.float64), yr, sr, "f32", f"replay {k}")
        call()                                       # an ordinary call between the replays
        torch.cuda.synchronize()
        assert_close(y.cpu().numpy().astype(np.float64), yr, sr, "f32", f"call {k}")
    P.pconv_get_async_error(h)
    h.free()
