"""The workspace's rest-pass sections where the pair capacity leaves no room for a rest pass (and its
launches are left out): the tiles left open by the first pass, and a rest pass of no pairs, as with a
capacity that has room for one."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu


def sections(views, scene, room):
    import paper_2412_12734_amd as gb
    sp = gb.Splats.from_numpy(scene)
    rast = gb.Rasterizer(views)
    slots = 1024 * sum(-(-v.width // 16) * -(-v.height // 16) for v in views)
    rast.plan(sp, slots + 5000 if room else slots)
    rast.ws.fill_(0xA5)
    rgb, T = rast.forward(sp)
    lay, n = rast.layout, rast.layout.total_tiles
    assert (lay.pair_capacity > lay.prefix_capacity) == room and not rast.status()[1]
    get = lambda name, k: rast.section(name, k).cpu().numpy().view(np.uint32)
    return dict(rgb=rgb, T=T, open=get("open_tiles", (n + 31) // 32),
                rest=get("ranges_rest", 2 * n), last=get("n_last_rest", rast.total_pixels))


def test_rest_sections_without_a_rest_pass():
    # dense enough that some tiles end, and views whose last tiles are cut
    scene = sg.make_scene(31, 3000, -0.7, 0.7, 0.05, 0.4, 4, op_lo=0.5, op_hi=0.95)
    views = [sg.look_at_view((0.0, 0.0, -3.5), 125, 90), sg.look_at_view((0.5, 0.3, -3.0), 72, 50)]
    want, got = sections(views, scene, True), sections(views, scene, False)
    assert torch.equal(got["rgb"], want["rgb"]) and torch.equal(got["T"], want["T"])
    bits = np.unpackbits(want["open"].view(np.uint8), bitorder="little")
    tiles = len(want["rest"]) // 2
    assert 0 < bits[:tiles].sum() < tiles
    np.testing.assert_array_equal(got["open"], want["open"])
    np.testing.assert_array_equal(want["rest"], 0)
    np.testing.assert_array_equal(got["rest"], 0)
    base = tile0 = 0
    for v in views:
        tx = -(-v.width // 16)
        y, x = np.divmod(np.arange(v.width * v.height), v.width)
        on = bits[tile0 + y // 16 * tx + x // 16].astype(bool)
        for s in (want, got):
            np.testing.assert_array_equal(s["last"][base:base + v.width * v.height][on], 0)
        base, tile0 = base + v.width * v.height, tile0 + tx * -(-v.height // 16)
