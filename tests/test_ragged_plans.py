"""Tiles of networks on odd maps: rows of no multiple of 4 pixels are staged in vectors and planned as such."""
import ctypes
import re

import pytest

import pb_workloads as W
from paper_2003_11666_amd.binding import plan_summary


@pytest.mark.parametrize("hw,layers,groups", [(146, (1, 3, 1, 3), 32), (165, (2, 4, 2), 16), (195, (2, 2, 5), 16)])
def test_strided_shortcuts_on_odd_maps_are_few_tiles(hw, layers, groups):
    """512 to 1024 channels, stride 2: 448 to 704 tiles of 16 x 16 forward if an element cost what a vector does."""
    net = W._net("odd", W.preact_resnet_bottleneck(layers, 64, groups, n_classes=19), 3, hw, hw, 19, 1e-3, 0.9, 8, 3, 8)
    steps = [l for l in plan_summary(net).splitlines() if re.search(r"C512x\d+x\d+ K1024x\d+x\d+ k1 s2 \| gm1", l)]
    assert len(steps) == 1 and int(re.search(r"tiles +(\d+)", steps[0])[1]) <= 256 and "tile 16x16" not in steps[0], steps


def test_the_first_layers_gradient_keeps_its_shares():
    """32 channels at 127 pixels: more, shorter shares than vectors alone would have it."""
    net = W._net("stem", W.preact_resnet_bottleneck((1, 3, 6, 1), 32, 16, n_classes=76), 3, 127, 127, 76, 1e-3, 0.9, 8, 3, 8)
    steps = [l for l in plan_summary(net).splitlines() if "C3x127x127" in l and "gm3" in l]
    assert len(steps) == 1 and int(re.search(r"tiles +(\d+)", steps[0])[1]) >= 96, steps


@pytest.mark.parametrize("hw", [(7, 7), (6, 6), (5, 8), (14, 14)])
@pytest.mark.parametrize("budget", [-1.0, 14.0])
def test_many_small_groups_are_planned_with_non_temporal_stores_asked_for(hw, budget):
    """33 groups of 4 channels in 17 layers: a wavefront takes a group's statistics on maps of no multiple of 4 pixels too."""
    from paper_2003_11666_amd import binding as B
    st = [[W.conv(3, 132, 1, 1, 0)]] + [[W.gn(33, 132), W.relu(), W.conv(132, 132, 1, 1, 0)] for _ in range(16)]
    st.append([W.gn(33, 132), W.relu(), W.gap(), W.linear(132, 5), W.ce()])
    desc, keep = B.marshal_net(W._net("groups", st, 3, *hw, 5, 1e-3, 0.9, 8, 3, 8), tuning=dict(tile_budget_us=budget, nt_stores=1))
    lib = B.load_library()
    assert lib.pb_arena_bytes(ctypes.byref(desc), None) > 0, lib.pb_last_error()


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("hw", range(4, 13))
def test_projections_beside_a_layer_behind_a_relu_are_planned(hw, stride):
    """The layer's own rows are rectified on their way into LDS, element by element; the skip tensor's come in vectors."""
    from paper_2003_11666_amd import binding as B
    st = [[W.conv(3, 5, 3, 1, 1)], [W.relu(), W.conv(5, 7, 3, stride, 1)], [W.relu(), W.conv(7, 7, 3, 1, 1), W.add(1, 5, 7, stride, 1)],
          [W.gn(1, 7), W.relu(), W.gap(), W.linear(7, 5), W.ce()]]
    lib = B.load_library()
    for tuning in (None, dict(tile_budget_us=14.0)):
        desc, keep = B.marshal_net(W._net("projection", st, 3, hw, hw, 5, 1e-3, 0.9, 8, 3, 8), tuning=tuning)
        assert lib.pb_arena_bytes(ctypes.byref(desc), None) > 0, lib.pb_last_error()


@pytest.mark.parametrize("width", [24, 48])
def test_rows_of_one_pixel_are_no_more_chunks_for_their_vectors(width):
    """3x3 layers of 8 x width channels on 1x1 maps: as many channels per chunk as LDS holds element by element."""
    from perf.cases import _network, _train
    net = _network(_train(None, "vgg", 0, hw=6, width=width, groups=8))
    c = 8 * width
    steps = [l for l in plan_summary(net).splitlines() if re.search(rf"C{c}x1x1 K{c}x1x1 k3 s1 \| gm[12]", l)]
    assert len(steps) >= 4, steps
    assert all(int(re.search(r"chunks (\d+)/", l)[1]) == width // 12 for l in steps), steps


def test_statistics_start_by_how_long_their_form_takes():
    """24 642 elements of a map of no multiple of 4 pixels, in three passes over memory, ahead of 12 800 elements of 512 channels by way
    of LDS, and those ahead of as many in registers."""
    st = [[W.conv(3, 36, 3, 1, 1)], [W.gn(2, 36), W.relu(), W.conv(36, 512, 1, 8, 0)], [W.gn(1, 512), W.relu(), W.conv(512, 512, 1, 1, 0)],
          [W.gn(4, 512), W.relu(), W.conv(512, 8, 1, 1, 0)], [W.gn(1, 8), W.relu(), W.gap(), W.linear(8, 5), W.ce()]]
    plan = plan_summary(W._net("stats", st, 3, 37, 37, 5, 1e-3, 0.9, 8, 3, 8), tuning=dict(tile_budget_us=16.0))
    order = [(m[2], m[1]) for m in re.finditer(r"phase (\d+) gn_stats .* C(\d+x\d+x\d+) ", plan)]
    assert order == [("36x37x37", "0"), ("512x5x5", "0"), ("512x5x5", "0")], order
    stages = [int(m[1]) for m in re.finditer(r"stage +(\d+) phase 0 gn_stats", plan)]
    assert stages == [1, 2, 3], stages
