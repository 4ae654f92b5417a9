"""The blend variants that the number of tiles chooses, where small test images do not reach them:
lists at the edges of the backward's short passes (32 entries with 8 x 8 grids, 48 with 16 x 16, both
on many tiles only), grids of several sides and view-dependent colour at every batch size, and the
forward's longest-lists-first order at both of its limits. Against the oracle on a crop."""
import numpy as np
import pytest
import torch

import scenegen as sg
from oracle import gb_oracle as O
from test_gpu_parity import assert_decreasing_in_buckets, check_grads, gb, gpu_opts  # noqa: F401

pytestmark = pytest.mark.gpu

# 225, 289, 625, 900, 1517, 1681 and 2401 tiles
SIZES = [(240, 240), (272, 272), (400, 400), (480, 480), (656, 592), (656, 656), (784, 784)]


def centre(size):
    return (size[0] // 2 - 24, size[1] // 2 - 20, 48, 40)


@pytest.mark.parametrize("N", [8, 16])
@pytest.mark.parametrize("P", [31, 32, 33, 47, 48, 49, 63, 64, 65, 97])
def test_lists_at_the_edges_of_a_short_pass(gb, N, P):  # noqa: F811
    size = SIZES[-1]
    scene = sg.make_scene(500 + P, P, -0.01, 0.01, 0.001, 0.012, N, op_lo=0.05, op_hi=0.3)
    view = sg.look_at_view((0.0, 0.0, -2.0), *size)
    rast = gb.Rasterizer([view])
    rast.forward(gb.Splats.from_numpy(scene))
    assert rast.layout.total_tiles == 2401
    ranges = rast.section("ranges", 2 * 2401).cpu().numpy().reshape(-1, 2)
    assert (ranges[:, 1] - ranges[:, 0]).max() == P
    check_grads(gb, scene, view, O.Options(), centre(size), seed=P)


@pytest.mark.parametrize("layout,sides", [(8, (1, 3, 8)), (16, (2, 5, 16))])
@pytest.mark.parametrize("size", SIZES)
def test_grids_of_several_sides_by_the_number_of_tiles(gb, layout, sides, size):  # noqa: F811
    scene = sg.make_scene(18, 150, -0.1, 0.1, 0.002, 0.1, 2, op_lo=0.02, op_hi=0.2)
    scene = sg.with_mixed_sides(scene, 4, sides)
    view = sg.look_at_view((0.05, 0.02, -2.0), *size)
    check_grads(gb, scene, view, O.Options(), centre(size), seed=layout)


@pytest.mark.parametrize("N", [1, 4, 8, 16])
@pytest.mark.parametrize("size", SIZES[::2])
def test_view_dependent_colour_by_the_number_of_tiles(gb, N, size):  # noqa: F811
    scene = sg.make_scene(19, 120, -0.1, 0.1, 0.002, 0.1, N, op_lo=0.02, op_hi=0.2)
    scene = sg.with_sh(scene, 5, 2, scale=0.3)
    view = sg.look_at_view((0.05, 0.02, -2.0), *size)
    check_grads(gb, scene, view, O.Options(bg=(0.1, 0.2, 0.3)), centre(size), seed=N)


@pytest.mark.parametrize("size,tiles,ordered", [((512, 384), 768, False), ((400, 496), 775, True),
                                                ((1280, 1024), 5120, True),
                                                ((1152, 1137), 5184, False)])
def test_forward_takes_the_longest_lists_first(gb, size, tiles, ordered):  # noqa: F811
    scene = sg.make_scene(23, 400, -0.6, 0.6, 0.002, 0.2, 4, op_lo=0.05, op_hi=0.6)
    views = [sg.look_at_view((0.05, 0.02, -2.0), *size)]
    out = []
    for order in (1, -1):
        o = gpu_opts(O.Options())
        o.tile_order = order
        sp = gb.Splats.from_numpy(scene)
        rast = gb.Rasterizer(views, o)
        rast.plan(sp)
        assert rast.layout.total_tiles == tiles
        rast.ws.fill_(0xA5)
        out.append(rast.forward(sp))
        if order == 1:
            took = rast.section("tile_order", tiles).cpu().numpy().view(np.uint32)
            if ordered:
                np.testing.assert_array_equal(np.sort(took), np.arange(tiles))
                r = rast.section("ranges", 2 * tiles).cpu().numpy().reshape(-1, 2).astype(np.int64)
                assert_decreasing_in_buckets((r[:, 1] - r[:, 0])[took])
            else:
                assert np.all(took == 0xA5A5A5A5)
    (rgb0, T0), (rgb1, T1) = out
    assert float(T0.min()) < 0.5
    assert torch.equal(rgb0, rgb1) and torch.equal(T0, T1)
