"""Waves on their own in workgroups of eight and four waves (fp32 NCHW): every shift of the last patch of a row in tiles of
whole rows and in tiles that cut rows, waves without a channel, strides 1 and 2, the fused max-pool."""
import numpy as np
import pytest

import oracle
import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, make_input, make_layer

from gpu_util import assert_close, say, to_device

pytestmark = pytest.mark.gpu

# (n, c_in, c_out, h, w)
WHOLE = [(1, 1, 4, 4, 4), (3, 17, 9, 5, 7), (2, 40, 6, 9, 60), (1, 33, 5, 14, 14), (5, 3, 8, 7, 9), (1, 70, 4, 13, 256), (9, 24, 70, 28, 28)]
CUT = [(1, 9, 5, 6, 260), (1, 9, 5, 6, 259), (1, 9, 5, 6, 262), (2, 9, 5, 6, 261)]


@pytest.fixture(autouse=True)
def _reset():
    yield
    P.pconv_debug_set_tiling(0, -1, -1)
    P.pconv_set_kernel_policy(0)


@pytest.mark.parametrize("waves,ks", [(8, 6), (4, 7)])
@pytest.mark.parametrize("shape,cut", [(s, 0) for s in WHOLE] + [(s, 1) for s in CUT])
def test_small_workgroups(shape, cut, waves, ks):
    import torch
    n, ci, co, h, w = shape
    P.pconv_set_kernel_policy(2)
    for dense in (False, True):
        spec = LayerSpec("wg", n, ci, co, h, w, num_patterns=1 if dense else 12, pattern_dist="dense" if dense else "uniform",
                         keep_div=2.0, count_dist="bernoulli")
        L = make_layer(spec, 6200 + w); x = make_input(spec, 6200 + w)
        hd = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
        P.pconv_debug_set_tiling(16, ks, -1)
        xd = to_device(x, "f32"); b = torch.from_numpy(L["bias"]).cuda()
        wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
        for stride in (1, 2):
            plan = P.pconv_debug_plan(hd, n, h, w, stride)
            assert (plan.waves, plan.ks_log2, plan.lone_cut) == (waves, 4, cut)
            say(f"[case] small workgroups {shape} waves={waves} stride={stride} dense={dense}")
            y = P.conv2d(hd, xd, b, stride=stride, relu=bool(n & 1))
            torch.cuda.synchronize()
            yr, sr = oracle.conv2d(x, wt, L["bias"], stride=stride, pad=1, relu=bool(n & 1))
            assert_close(y.cpu().numpy().astype(np.float64), yr, sr, "f32", f"wg{shape} stride {stride}")
        if w % 2 == 0:
            say(f"[case] small workgroups {shape} waves={waves} pool dense={dense}")
            y = P.conv2d_pool2x2(hd, xd, b)
            y2 = P.maxpool2x2(P.conv2d(hd, xd, b))
            torch.cuda.synchronize()
            assert torch.equal(y, y2)
        hd.free()


# (n, c_in, c_out, h, w): widths 1, 2 and 3 beyond a multiple of 4, rows of fewer and of more than 64 patches
PARTED = [(4, 24, 24, 42, 129), (4, 24, 24, 42, 130), (5, 24, 24, 33, 146), (3, 24, 24, 95, 139), (5, 24, 16, 21, 274)]


@pytest.mark.parametrize("form", ["plain", "stride2", "pool"])
@pytest.mark.parametrize("waves,ks", [(16, 4), (16, 5), (8, 6), (4, 7)])
@pytest.mark.parametrize("shape", PARTED)
def test_equal_images_get_equal_outputs(shape, waves, ks, form):
    """Tiles that cut rows, one of which ends between the last two patches of a row: both workgroups store the columns
    that these share.  With stride 2 and an even width the stored outputs have a loop and a sum of their own."""
    import torch
    n, ci, co, h, w = shape
    if form == "pool" and w % 2:
        pytest.skip("the fused pool takes even widths")
    px, stride = (w + 3) // 4, 2 if form == "stride2" else 1
    per_image = (h + 3) // 4 * px
    spec = LayerSpec("wg", 1, ci, co, h, w)
    L = make_layer(spec, 6300 + w); x = make_input(spec, 6300 + w)
    hd = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32")
    P.pconv_debug_set_tiling(16, ks, -1)
    plan = P.pconv_debug_plan(hd, n, h, w, stride, fuse_pool=form == "pool")
    assert (plan.waves, plan.ks_log2, plan.lone_cut, plan.lone_patches) == (waves, 5 if ks == 5 else 4, 1, 64)
    assert w % 4 and per_image % 64 and any(64 * k % px == px - 1 for k in range(1, (n * per_image + 63) // 64))
    say(f"[case] equal images {shape} waves={waves} ks={ks} {form}")
    xd = to_device(x, "f32").repeat(n, 1, 1, 1)
    ys = [P.conv2d_pool2x2(hd, xd) if form == "pool" else P.conv2d(hd, xd, stride=stride) for _ in range(4)]
    torch.cuda.synchronize()
    assert all(torch.equal(y, ys[0]) for y in ys) and torch.equal(ys[0], ys[0][:1].expand_as(ys[0]))
    if form != "pool":
        wt = oracle.masked_weights(L["w"], L["pattern_id"], L["conn"], L["table"])
        yr, sr = oracle.conv2d(x, wt, None, stride=stride, pad=1)
        assert_close(ys[0][:1].cpu().numpy().astype(np.float64), yr, sr, "f32", f"equal{shape} {form}")
    hd.free()
