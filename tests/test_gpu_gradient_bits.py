"""The record gradients to the last bit. Sums that make up a scale's gradient can cancel (exactly
so where the falloff is the screen low-pass's and one coordinate is clamped to the grid's border),
and Adam's first steps divide a gradient by its own size: another rounding of such a sum moves the
parameter by a full step the other way, so that a training run changes. The bits are those of the
kernels before the backward was rearranged; every splat here touches one or two 8 x 8 blocks, so
that no sum depends on an order of arrival (a + b is b + a)."""
import zlib

import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu

W, H, F = 96, 80, 80.0
ARRAYS = ("means", "tan_u", "tan_v", "scales", "opacity")
# CRC-32 of each array's bytes
BITS = {
    "1 f32": (0x2a292a44, 0x14a8d4d9, 0x821c2ceb, 0x65779968, 0x70c42abf),
    "2 f32": (0x67ea707a, 0xfe8d1888, 0x5a2441f9, 0xa74531f6, 0x03d0acc2),
    "4 f32": (0x474b1592, 0x6525a285, 0xb48d55e0, 0x889ed422, 0x3dfa9b33),
    "4 bf16": (0x2754919c, 0xce5b2603, 0x797f11f3, 0x2920a99d, 0xff5250bb),
    "8 f32": (0x87c303a4, 0x117aca03, 0x85a96963, 0x86c28917, 0xa9b901ac),
    "16 f32": (0x6d4a4bbf, 0xf23ebec9, 0x2a245f92, 0xb5a4a3ce, 0x7124227a),
    "8 1,3,8": (0xf6d9b1c7, 0xd81aea25, 0x7d3ebf21, 0x7da09587, 0x9657e595),
    "16 1,5,16": (0x7978d367, 0x2eabc23e, 0xb751cc43, 0x4cbde38d, 0x59a32cab),
}


def block_scene(N, sides=None):
    """Three layers of splats over every 8 x 8 block, 0.02 to 0.85 pixels wide (thin and edge-on
    ones among them), inside the block or, every other one of the last layer, across its left edge."""
    rng = np.random.default_rng(11)
    by, bx, layer = (a.reshape(-1) for a in np.meshgrid(np.arange(H // 8), np.arange(1, W // 8),
                                                        np.arange(3), indexing="ij"))
    P = len(bx)
    z = 2.0 + 0.01 * rng.permutation(P) / P + 0.1 * layer
    edge = (layer == 2) & ((bx + by) % 2 == 0)
    px = 8 * bx + np.where(edge, 0, 4) + rng.uniform(-0.5, 0.5, P)
    py = 8 * by + 4 + rng.uniform(-0.5, 0.5, P)
    means = np.stack([(px - W / 2) / F * z, (py - H / 2) / F * z, z], 1)
    q = rng.standard_normal((P, 4))
    q[::3, 1:3] = 0.0  # a third of them face the camera
    q /= np.sqrt((q * q).sum(1, keepdims=True))
    w, x, y, t = q.T
    tan_u = np.stack([1 - 2 * (y * y + t * t), 2 * (x * y + w * t), 2 * (x * t - w * y)], 1)
    tan_v = np.stack([2 * (x * y - w * t), 1 - 2 * (x * x + t * t), 2 * (y * t + w * x)], 1)
    size = np.array([0.02, 0.1, 0.4, 0.85])[rng.integers(0, 4, (P, 2))] * rng.uniform(0.9, 1.0, (P, 2))
    f = lambda a: np.ascontiguousarray(a, dtype=np.float32)
    if sides:
        tex = [f(rng.uniform(0, 1, (n, n, 3))) for n in rng.choice(sides, P)]
    else:
        tex = f(rng.uniform(0, 1, (P, N, N, 3)))
    return sg.Scene(f(means), f(tan_u), f(tan_v), f(size * z[:, None] / F),
                    f(rng.uniform(0.3, 0.95, P)), tex)


@pytest.mark.parametrize("batch_bwd", [0, 8])
@pytest.mark.parametrize("case", sorted(BITS))
def test_record_gradients_keep_their_bits(case, batch_bwd):
    import paper_2412_12734_amd as gb
    layout, kind = case.split()
    N = int(layout)
    sides = [int(s) for s in kind.split(",")] if "," in kind else None
    sp = gb.Splats.from_numpy(block_scene(N, sides), tex_bf16=kind == "bf16")
    view = sg.View(width=W, height=H, fx=F, fy=F, cx=W / 2, cy=H / 2,
                   R=np.eye(3, dtype=np.float32), t=np.zeros(3, np.float32), z_near=0.01)
    rast = gb.Rasterizer([view], gb.Options(batch_bwd=0 if N == 16 else batch_bwd))
    g = torch.from_numpy(np.random.default_rng(12).choice(
        np.float32([-1, 1]) / np.float32(3 * W * H), (W * H, 3))).cuda()
    rgb, T = rast.forward(sp)
    grads = rast.backward(sp, T, g)
    got = {k: zlib.crc32(grads[k].cpu().numpy().tobytes()) for k in ARRAYS}
    assert float(grads["scales"].abs().max()) > 0
    assert got == dict(zip(ARRAYS, BITS[case]))
