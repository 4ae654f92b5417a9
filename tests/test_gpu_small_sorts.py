"""The one-launch depth order, pair scan and pair sort of small calls at the edges of their ranges,
against the oracle's pair lists: record counts around a wave's, a workgroup's and the largest that
takes them, equal depths (ties go by record index), culled records, images whose tiles take one
sort pass and two, and pair slots on both sides of the one-launch sort's."""
import numpy as np
import pytest
import torch

import scenegen as sg
from oracle import gb_oracle as O
from test_gpu_parity import gb, run_gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(40, 24), (300, 290)])  # 6 and 361 tiles
@pytest.mark.parametrize("P,views", [(1, 1), (63, 1), (64, 1), (65, 1), (1024, 1), (1025, 1),
                                     (4095, 2), (5461, 3), (8192, 2), (8193, 2), (12288, 2),
                                     (24577, 1)])
def test_pair_lists_match_the_oracle(gb, P, views, size):  # noqa: F811
    scene = sg.make_scene(P, P, -1.2, 1.2, 0.001, 0.02, 2, op_lo=0.02, op_hi=0.2)
    if P > 4:  # equal depths: the same centre, rotation and scales at other indices
        for a in (scene.means, scene.tan_u, scene.tan_v, scene.scales):
            a[P // 2] = a[1]
            a[P - 1] = a[1]
    # the second view looks away from most of the scene (culled records)
    eyes = [(0.05, 0.02, -2.0), (0.3, 0.1, 0.2), (1.0, -0.4, -2.5)]
    vs = [sg.look_at_view(e, *size) for e in eyes[:views]]
    opts = O.Options()
    # (prefix slots for every pair: the first pass holds the whole list)
    rast, _, rgb, T = run_gpu(gb, scene, vs, opts, prefix=8192)
    keys, vals, _ = O.tile_pairs(scene, vs, opts)
    n = len(keys)
    st = rast.section("status", 8).cpu().numpy().view(np.uint32)
    assert int(st[0]) == n and int(st[1]) == n and int(st[2]) == 0
    gk = rast.section("pair_keys", n).cpu().numpy().view(np.uint32)
    gv = rast.section("pair_vals", n).cpu().numpy().view(np.uint32)
    np.testing.assert_array_equal(gk, keys)
    np.testing.assert_array_equal(gv, vals)
    tiles = rast.layout.total_tiles
    r = rast.section("ranges", 2 * tiles).cpu().numpy().view(np.uint32).reshape(-1, 2)
    first = np.searchsorted(keys, np.arange(tiles), "left")
    end = np.searchsorted(keys, np.arange(tiles), "right")
    np.testing.assert_array_equal(r[:, 1] - r[:, 0], end - first)
    np.testing.assert_array_equal(r[end > first, 0], first[end > first])
    # a split into prefix and rest passes gives the same image bit for bit
    _, _, rgb1, T1 = run_gpu(gb, scene, vs, opts, prefix=1)
    assert torch.equal(rgb, rgb1) and torch.equal(T, T1)
