"""The form that a call of the register-tiled kernel (fp32 NCHW) takes, for layers where another one was measured slower."""
import pytest

import paper_1909_05073_amd as P
from pconv_inputs import LayerSpec, make_layer


def plan_of(shape, keep, pool=False):
    """(waves of a workgroup, ks_log2, split_units) on 256 compute units."""
    n, ci, co, h, w, stride = shape
    L = make_layer(LayerSpec("plan", 1, ci, co, 8, 8, stride=stride, keep_div=keep), 8100 + ci)
    hd = P.pconv_pack(L["w"], L["pattern_id"], L["conn"], L["table"], "f32", host_only=True)
    p = P.pconv_debug_plan(hd, n, h, w, stride, fuse_pool=pool)
    hd.free()
    assert p.kernel == 2
    return p.waves, p.ks_log2, p.split_units


# ((n, c_in, c_out, h, w, stride), keep, us with two slots, us with four slots and the best number of waves)
TWO_SLOTS = [((27, 11, 44, 12, 14, 1), 2.5, 4.9, 5.9), ((2, 24, 329, 19, 19, 1), 8.0, 4.8, 6.0), ((1, 11, 69, 39, 46, 1), 2.5, 4.8, 5.8),
             ((6, 8, 8, 23, 25, 1), 1.5, 4.6, 5.4), ((3, 6, 18, 29, 29, 2), 1.5, 4.3, 5.2), ((2, 29, 10, 16, 16, 1), 8.0, 4.2, 5.3)]


@pytest.mark.parametrize("shape,keep,two,four", TWO_SLOTS)
def test_small_layers_take_two_slots_a_workgroup(shape, keep, two, four):
    assert two < 0.9 * four and plan_of(shape, keep)[:2] == (16, 5)


# (..., waves, us, us with two slots)
FOUR_SLOTS = [((30, 325, 46, 29, 31, 1), 8.0, 8, 22.5, 25.2), ((1, 160, 44, 200, 160, 1), 2.5, 8, 28.9, 31.9),
              ((24, 31, 330, 26, 20, 1), 3.6, 4, 18.3, 42.0), ((9, 38, 47, 104, 124, 2), 1.5, 4, 19.8, 46.8)]


@pytest.mark.parametrize("shape,keep,waves,four,two", FOUR_SLOTS)
def test_larger_ones_keep_four(shape, keep, waves, four, two):
    assert four < 0.95 * two and plan_of(shape, keep)[:2] == (waves, 4)


# (..., us of the whole or shared units taken, us of workgroups of 4 waves on their own)
BEYOND_L2 = [((36, 491, 63, 79, 82, 2), 3.6, 254, 603), ((5, 385, 44, 165, 200, 1), 3.6, 165, 318), ((7, 368, 50, 181, 182, 1), 8.0, 152, 244),
             ((62, 149, 50, 82, 98, 2), 2.5, 152, 245), ((16, 256, 47, 152, 152, 1), 2.5, 272, 425)]


@pytest.mark.parametrize("shape,keep,units,lone", BEYOND_L2)
def test_tiles_beyond_the_l2_are_not_read_by_every_block_of_filters(shape, keep, units, lone):
    assert units < 0.95 * lone and plan_of(shape, keep)[1] < 4


# (..., us with 4 waves on their own, us of whole units)
WITHIN_L2 = [((4, 113, 110, 117, 141, 1), 8.0, 35.1, 51.0), ((12, 61, 402, 42, 34, 1), 3.6, 31.8, 42.7), ((23, 173, 385, 26, 29, 1), 3.6, 70.8, 102.4)]


@pytest.mark.parametrize("shape,keep,lone,units", WITHIN_L2)
def test_others_are(shape, keep, lone, units):
    assert lone < 0.95 * units and plan_of(shape, keep)[:2] == (4, 4)


# (..., us of whole units, us of workgroups of 4 waves on their own): waves of a unit without filters; stride 2 with an even width
IDLE_OR_QUARTER = [((37, 32, 35, 204, 207, 1), 3.6, 143, 178), ((41, 10, 75, 134, 160, 1), 3.6, 101, 118), ((52, 82, 30, 185, 148, 1), 2.5, 270, 327),
                   ((8, 200, 460, 64, 64, 2), 2.5, 103, 127), ((44, 170, 153, 87, 88, 2), 2.5, 328, 395), ((28, 332, 502, 49, 58, 2), 3.6, 420, 485)]


@pytest.mark.parametrize("shape,keep,units,lone", IDLE_OR_QUARTER)
def test_units_with_idle_waves_or_a_quarter_of_the_outputs(shape, keep, units, lone):
    assert units < 0.95 * lone and plan_of(shape, keep)[1] < 4


# (..., us of whole units, us of workgroups of 4 waves on their own), the max-pool fused
POOLED = [((5, 10, 144, 172, 206, 1), 8.0, 25.9, 32.6), ((1, 5, 429, 118, 140, 1), 3.6, 10.7, 13.2), ((2, 16, 118, 175, 176, 1), 3.6, 14.5, 17.8),
          ((32, 18, 46, 214, 170, 1), 8.0, 59.4, 72.4), ((16, 7, 123, 54, 64, 1), 3.6, 10.1, 12.1)]


@pytest.mark.parametrize("shape,keep,units,lone", POOLED)
def test_units_that_store_pooled_outputs(shape, keep, units, lone):
    assert units < 0.95 * lone and plan_of(shape, keep, pool=True)[1] < 4


def test_pooled_layers_of_many_channels_stay_on_their_own():
    assert plan_of((32, 512, 512, 14, 14, 1), 3.6, pool=True)[:2] == (4, 4)
