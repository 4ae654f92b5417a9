"""The blend's staging passes and texel groups at their edges, against the oracle: lists that end
one short of, at and one past a pass of 64 entries (32 in the backward of 16 x 16 grids) and
splats that touch a tile without reaching it; grids of side 1, 2 (no clamped end is inferred), 3
and up; thin and sub-pixel splats, whose falloff is the low-pass's."""
import numpy as np
import pytest
import torch

import scenegen as sg
from oracle import gb_oracle as O
from test_gpu_parity import check_grads, gb, gpu_opts, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("P", [1, 31, 32, 33, 63, 64, 65, 128, 129])
def test_lists_at_the_edges_of_a_pass(gb, N, P):  # noqa: F811
    scene = sg.make_scene(300 + P, P, -0.3, 0.3, 0.002, 0.3, N, op_lo=0.02, op_hi=0.2)
    view = sg.look_at_view((0.05, 0.02, -2.0), 37, 29)
    opts = O.Options()
    _, _, rgb, T = run_gpu(gb, scene, [view], opts)
    if N < 16:  # other batches cut the passes elsewhere: the same image bit for bit
        _, _, rgb1, T1 = run_gpu(gb, scene, [view], opts, batch=8)
        assert torch.equal(rgb, rgb1) and torch.equal(T, T1)
    check_grads(gb, scene, view, opts, (0, 0, 37, 29), seed=P)


@pytest.mark.parametrize("N", [2, 4, 8, 16])
@pytest.mark.parametrize("size", [(272, 272), (400, 400), (480, 480), (656, 592)])
def test_batches_by_the_number_of_tiles(gb, N, size):  # noqa: F811
    # 289, 625, 900 and 1517 tiles: how many run at once decides the batch sizes
    scene = sg.make_scene(17, 150, -0.1, 0.1, 0.002, 0.1, N, op_lo=0.02, op_hi=0.2)
    view = sg.look_at_view((0.05, 0.02, -2.0), *size)
    crop = (size[0] // 2 - 24, size[1] // 2 - 20, 48, 40)
    check_grads(gb, scene, view, O.Options(), crop, seed=N)


@pytest.mark.parametrize("size", [(448, 432), (448, 449), (1139, 1145), (1152, 1137)])
def test_forward_tile_order_changes_no_pixel(gb, size):  # noqa: F811
    # 756, 812, 5184 and 5112 tiles: on both sides of the numbers that are walked longest list first
    scene = sg.make_scene(23, 400, -0.6, 0.6, 0.002, 0.2, 4, op_lo=0.05, op_hi=0.6)
    views = [sg.look_at_view((0.05, 0.02, -2.0), *size)]
    out = []
    for order in (1, -1):
        o = gpu_opts(O.Options())
        o.tile_order = order
        sp = gb.Splats.from_numpy(scene)
        rast = gb.Rasterizer(views, o)
        rast.plan(sp)
        out.append(rast.forward(sp))
    (rgb0, T0), (rgb1, T1) = out
    assert float(T0.min()) < 0.5
    assert torch.equal(rgb0, rgb1) and torch.equal(T0, T1)


@pytest.mark.parametrize("layout,sides", [(8, (1, 2, 3, 8)), (16, (1, 2, 5, 16))])
def test_thin_splats_with_grids_of_several_sides(gb, layout, sides):  # noqa: F811
    scene = sg.make_scene(7, 200, -0.5, 0.5, 0.001, 0.4, 2)
    scene.scales[:, 0] = np.minimum(scene.scales[:, 0], 0.004)
    scene = sg.with_mixed_sides(scene, 3, sides)
    view = sg.look_at_view((0.1, -0.1, -2.5), 50, 41)
    check_grads(gb, scene, view, O.Options(), (0, 0, 50, 41), seed=2)
