"""When conv2d lends a call with channels last work space out of torch's allocator, and when it must not."""
import ctypes as C
from types import SimpleNamespace

import numpy as np
import pytest

import oracle
import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, make_input, make_layer

from gpu_util import assert_close, say


class FakeLibrary:
    """Asks for work space and notes what it is lent."""

    def __init__(self):
        self.lent, self.mode, self.knows_modes = [], 0, True
        self.asks, self.calls = 4096, []

    def pconv_conv2d_workspace(self, *call):
        self.calls.append("workspace")
        return self.asks

    def pconv_conv2d_or_workspace(self, *call):
        self.calls.append("or_workspace")
        return self.asks

    def pconv_conv2d_ws(self, *call):
        self.calls.append("ws")
        self.lent.append(call[-2:])
        return P.OK

    def hipThreadExchangeStreamCaptureMode(self, mode):
        if not self.knows_modes:
            return 1
        self.mode, mode._obj.value = mode._obj.value, self.mode
        return 0


@pytest.fixture
def binding(monkeypatch):
    """The binding over a library that only takes notes, with tensors in host memory."""
    import torch
    fake = FakeLibrary()
    monkeypatch.setattr(P, "_lib", fake)
    monkeypatch.setattr(P, "_stream", lambda index: None)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    x = torch.zeros((1, 8, 8, 64))

    def call():
        out = torch.zeros((1, 8, 8, 64))
        assert P._conv2d_ws(SimpleNamespace(ptr=1, c_in=64), x, None, 1, False, out, 1, 8, 8) is out
        return fake.lent.pop()
    call.library = fake
    return call, monkeypatch, torch


def test_ordinary_calls_are_lent_what_they_ask_for(binding):
    call, _, _ = binding
    ptr, size = call()
    assert ptr and size == 4096


def test_small_layers_are_one_call_of_the_library(binding):
    """Asking first and calling then cost layers that use no work space a sixth of their time on the host."""
    import torch
    call, _, _ = binding
    fake = call.library
    x = out = torch.zeros((1, 8, 8, 8))
    small = lambda: P._conv2d_ws(SimpleNamespace(ptr=1, c_in=8), x, None, 1, False, out, 1, 8, 8)
    fake.asks = P.OK
    assert small() is out and len(fake.calls) == 1
    fake.asks = 4096                                 # (such a layer that does use it)
    assert small() is out and fake.lent.pop()[1] == 4096
    fake.asks, fake.pconv_last_error = P.INVALID_ARG, lambda: b"refused"
    with pytest.raises(P.PconvError):
        small()


def test_without_memory_for_it_the_call_goes_on_without(binding):
    call, monkeypatch, torch = binding

    def refuse(size, **kw):
        raise torch.cuda.OutOfMemoryError("no memory")
    monkeypatch.setattr(torch, "empty", refuse)
    assert call() == (None, 0)


@pytest.mark.parametrize("pool,lends", [((0, 0), False), ((3, 0), True), (None, False)])
def test_captured_calls_are_lent_memory_of_the_graph_or_none(binding, pool, lends):
    """None: the allocator does not tell its pools."""
    call, monkeypatch, torch = binding
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)

    def snapshot():
        if pool is None:
            raise RuntimeError("not supported")
        return [{"address": 0, "total_size": 1 << 62, "segment_pool_id": pool}]
    monkeypatch.setattr(torch.cuda, "memory_snapshot", snapshot)
    ptr, size = call()
    assert (bool(ptr), size) == ((True, 4096) if lends else (False, 0))


def test_the_allocator_is_asked_in_the_relaxed_mode_of_captures(binding):
    """It queries the events that it has outstanding, which makes a capture in another mode invalid."""
    call, monkeypatch, torch = binding
    empty, asked, pool = torch.empty, [], [(0, 0)]

    def note(size, **kw):
        asked.append((size, call.library.mode))
        return empty(size, **kw)
    monkeypatch.setattr(torch, "empty", note)
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: True)
    monkeypatch.setattr(torch.cuda, "memory_snapshot", lambda: [{"address": 0, "total_size": 1 << 62, "segment_pool_id": pool[0]}])
    assert call() == (None, 0) and asked == [(1, 2)] and call.library.mode == 0
    pool[0] = (3, 0)
    assert call()[1] == 4096 and asked == [(1, 2), (1, 2), (4096, 0)] and call.library.mode == 0

    def refuse(size, **kw):
        raise RuntimeError("refused")
    monkeypatch.setattr(torch, "empty", refuse)
    assert call() == (None, 0) and call.library.mode == 0
    call.library.knows_modes = False
    monkeypatch.setattr(torch, "empty", note)
    assert call() == (None, 0) and len(asked) == 3


@pytest.mark.gpu
def test_captures_of_torch_have_a_pool():
    import torch
    t = torch.zeros(8, device="cuda")
    g = torch.cuda.CUDAGraph()
    say("[case] capture by torch")
    with torch.cuda.graph(g):
        t.add_(1.0)
        served = P._graph_pool_serves(t.device)
    assert served and not P._graph_pool_serves(t.device)


@pytest.mark.gpu
@pytest.mark.parametrize("outstanding", [False, True])
def test_a_capture_that_torch_does_not_know_of(outstanding):
    """Captured with the HIP runtime alone, the output given: nothing of torch's ordinary pool may get into the graph,
    and the capture stays valid, also where torch's allocator has an event to query (outstanding)."""
    import torch
    L = P.lib()                                      # (the HIP runtime is a dependency of the library)

    def hip(name, *args):
        fn = getattr(L, name)
        fn.restype = C.c_int
        assert fn(*args) == 0, name
    n, ci, co, hh, ww = 2, 40, 200, 20, 24
    spec = LayerSpec("raw", n, ci, co, hh, ww, keep_div=2.5, count_dist="bernoulli")
    W = make_layer(spec, 7950)
    h = P.pconv_pack(W["w"], W["pattern_id"], W["conn"], W["table"], "f32")
    b = torch.from_numpy(W["bias"]).cuda()
    wt = oracle.masked_weights(W["w"], W["pattern_id"], W["conn"], W["table"])
    size = L.pconv_conv2d_workspace(h.ptr, n, hh, ww, 1, P.NHWC, P.F32)
    assert size > 0
    xs = torch.zeros((n, hh, ww, ci), device="cuda")
    ys = torch.empty((n, hh, ww, co), device="cuda")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        P.conv2d(h, xs, b, layout="nhwc", out=ys)
    torch.cuda.synchronize()
    say(f"[case] capture by the HIP runtime outstanding={outstanding}")
    st, graph, ready, state = C.c_void_p(side.cuda_stream), C.c_void_p(), C.c_void_p(), C.c_int()
    if outstanding:
        t = torch.zeros(1 << 20, device="cuda")
        other = torch.cuda.Stream()
        other.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(other):
            t.add_(1.0)
        t.record_stream(other)
        del t
    with torch.cuda.stream(side):
        hip("hipStreamBeginCapture", st, C.c_int(0))
        P.conv2d(h, xs, b, layout="nhwc", out=ys)
        hip("hipStreamIsCapturing", st, C.byref(state))
        assert state.value == 1                      # (active; 2: invalid)
        hip("hipStreamEndCapture", st, C.byref(graph))
    hip("hipGraphInstantiate", C.byref(ready), graph, None, None, C.c_size_t(0))
    # what the ordinary pool hands out next, on either stream: of the size that the call would have been lent
    mine = [torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(4)]
    with torch.cuda.stream(side):
        mine += [torch.full((size,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(4)]
    for k in range(3):
        xk = make_input(spec, 7951 + k)
        xs.copy_(torch.from_numpy(xk.transpose(0, 2, 3, 1).copy())); ys.fill_(float("nan"))
        torch.cuda.synchronize()
        hip("hipGraphLaunch", ready, st)
        torch.cuda.synchronize()
        yr, sr = oracle.conv2d(xk, wt, W["bias"], pad=1)
        assert_close(ys.permute(0, 3, 1, 2).cpu().numpy().astype(np.float64), yr, sr, "f32", f"replay {k}")
        assert all(bool((m == 0x5A).all()) for m in mine)
    hip("hipGraphExecDestroy", ready)
    hip("hipGraphDestroy", graph)
    h.free()


@pytest.mark.gpu
def test_more_images_than_a_transpose_has_workgroups():
    """A launch has fewer than 2^32 threads, and every image takes a workgroup of 256: 2^24 images are left to the
    kernel that takes them as they are, one fewer is the largest call that is lent work space."""
    import torch
    most, ci, co, hh, ww = (1 << 24) - 1, 5, 16, 1, 4      # (few channels are lent it where the output is most of the call)
    spec = LayerSpec("many", 64, ci, co, hh, ww, keep_div=1.5, count_dist="bernoulli")
    W = make_layer(spec, 7960)
    h = P.pconv_pack(W["w"], W["pattern_id"], W["conn"], W["table"], "f32")
    ask = lambda n: P.lib().pconv_conv2d_workspace(h.ptr, n, hh, ww, 1, P.NHWC, P.F32)
    assert ask(most + 1) == 0 and ask(1 << 25) == 0 and ask(most) > 0
    b = torch.from_numpy(W["bias"]).cuda()
    wt = oracle.masked_weights(W["w"], W["pattern_id"], W["conn"], W["table"])
    few = [make_input(spec, 7961 + k) for k in range(2)]
    x = torch.randn((most + 1, hh, ww, ci), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    for xk, part in zip(few, (x[:64], x[most - 64:most])):
        part.copy_(torch.from_numpy(xk.transpose(0, 2, 3, 1).copy()))
    ys = []
    for n in (most, most + 1):
        say(f"[case] {n} images of {ci} channels, {hh}x{ww}")
        ys.append(P.conv2d(h, x[:n], b, layout="nhwc"))
        torch.cuda.synchronize()
        for xk, part in zip(few, (ys[-1][:64], ys[-1][most - 64:most])):
            yr, sr = oracle.conv2d(xk, wt, W["bias"], pad=1)
            assert_close(part.permute(0, 3, 1, 2).cpu().numpy().astype(np.float64), yr, sr, "f32", f"{n} images")
    # at most 45 products in either order: 2 * 45 * 2^-24 of the sum of their sizes, which is below 100
    assert float((ys[0] - ys[1][:most]).abs().max()) < 1e-3
    h.free()
