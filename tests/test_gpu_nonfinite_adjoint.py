"""A pixel whose incoming adjoint is not finite (a loss that divided by zero) reaches the colours and
opacities of the splats that it blended and of no other: splats that share its 8 x 8 block without
touching it keep the gradients that they have with a zero adjoint there."""
import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu

W = H = 16


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("radius", [0.3, 3.0])  # pixels: a few of a block (one by one), or most (groups)
@pytest.mark.parametrize("N,sides", [(1, None), (2, None), (4, None), (8, None), (16, None),
                                     (8, (1, 2, 8))])
def test_other_splats_keep_their_colour_gradients(N, sides, radius, bad):
    import paper_2412_12734_amd as gb
    # splats seen face on by a camera at 1 pixel per unit and depth: six over pixel (15, 15), four
    # over (2, 2) of another block of the tile, and six in the first one's block away from it
    P = 16
    f = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    at = np.array([[15.5, 15.5]] * 6 + [[2.5, 2.5]] * 4 + [[10.4, 10.4]] * 6)
    s = np.where(np.arange(P) < 10, radius, min(radius, 1.3))[:, None] * np.ones((P, 2))
    z = 1.0 + 0.01 * np.arange(P)
    rng = np.random.default_rng(4)
    scene = sg.Scene(f(np.concatenate([at * z[:, None], z[:, None]], 1)),
                     f(np.tile([1, 0, 0], (P, 1))), f(np.tile([0, 1, 0], (P, 1))), f(s * z[:, None]),
                     f(np.full(P, 0.2)), f(rng.uniform(0.1, 1, (P, N, N, 3))))
    if sides:
        scene = sg.with_mixed_sides(scene, 3, sides)
    view = sg.View(width=W, height=H, fx=1.0, fy=1.0, cx=0.0, cy=0.0, R=np.eye(3, dtype=np.float32),
                   t=np.zeros(3, np.float32), z_near=0.01)
    sp = gb.Splats.from_numpy(scene)
    g = torch.ones((H * W, 3), device="cuda")
    pixel = 15 * W + 15
    out = []
    for value in (0.0, bad):
        g[pixel] = value
        rast = gb.Rasterizer([view])
        rgb, T = rast.forward(sp)
        out.append(rast.backward(sp, T, g.clone()))
    n = sp.n_texels // P if not sides else None
    first = (sp.tex_offset.cpu().numpy() if sides else np.arange(P) * n)
    rows = np.concatenate([[int(x) for x in first], [sp.n_texels]])
    t0, t1 = (o["textures"].reshape(-1, 3).cpu().numpy() for o in out)
    o0, o1 = (o["opacity"].cpu().numpy() for o in out)
    for k in range(P):
        a, b = t0[rows[k]:rows[k + 1]], t1[rows[k]:rows[k + 1]]
        if k < 6:
            assert not np.isfinite(b).all() and not np.isfinite(o1[k])
        else:
            assert np.abs(a).max() > 0
            # (sums over the blocks of a tile depend on an order of arrival)
            np.testing.assert_allclose(b, a, rtol=1e-5, atol=1e-5)
            assert abs(o1[k] - o0[k]) <= 1e-5 * abs(o0[k]) + 1e-5
