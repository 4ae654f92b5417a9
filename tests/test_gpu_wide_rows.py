"""The row gather of densification for rows of very many floats, which one workgroup would move one
after another: widths on both sides of where they are shared by all workgroups, among narrow ones,
against indexing."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

WIDTHS = (65535, 3, 65536, 65537, 12, 70004)


@pytest.mark.parametrize("shift", [0, 1])  # floats by which source and target are misaligned
@pytest.mark.parametrize("P", [1, 33, 67])
def test_state_rows_of_many_floats(P, shift):
    from paper_2412_12734_amd import _lib as L
    lib = L.load()
    rng = np.random.default_rng(P)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()
    # every third splat is transparent (pruned), every other of the rest is cloned
    k = np.arange(P)
    gone, clone = k % 3 == 2, k % 2 == 1
    src = dict(means=dev(rng.standard_normal((P, 3))), quats=dev(rng.standard_normal((P, 4))),
               log_scales=dev(np.full((P, 2), np.log(0.001))),
               opacity_logits=dev(np.where(gone, -9.0, 2.0)),
               textures=dev(rng.uniform(0, 1, (P, 2, 2, 3))))
    accum, vis = dev(np.where(clone, 1.0, 0.0)), dev(np.ones(P))
    noise = dev(np.zeros((P, 2, 2)))
    raw = lambda t, n: L.GbRawSplats(n, 2, 0, *(t[f].data_ptr() for f in (
        "means", "quats", "log_scales", "opacity_logits", "textures")), None)
    opts = L.GbDensifyOptions(2e-4, 0.01, 0.005, 0.0, 1.6)
    work = torch.empty(int(lib.gb_densify_work_bytes(P)), dtype=torch.uint8, device="cuda")
    n, stream = ctypes.c_int64(-1), torch.cuda.current_stream().cuda_stream
    L.check(lib.gb_densify_plan(ctypes.byref(raw(src, P)), accum.data_ptr(), vis.data_ptr(),
                                ctypes.byref(opts), work.data_ptr(), work.numel(),
                                ctypes.byref(n), stream), "plan")
    parent = np.concatenate([[i, i] if clone[i] else [i] for i in k if not gone[i]]).astype(int)
    new = np.concatenate([[0, 1] if clone[i] else [0] for i in k if not gone[i]]).astype(bool)
    n_new = len(parent)
    assert n.value == n_new
    out = {f: torch.full((n_new,) + tuple(t.shape[1:]), -7.0, device="cuda")
           for f, t in src.items()}
    ins = [dev(rng.standard_normal(shift + P * w)) for w in WIDTHS]
    outs = [torch.full((shift + n_new * w + 3,), -7.0, device="cuda") for w in WIDTHS]
    states = (L.GbRowState * len(WIDTHS))(*(
        L.GbRowState(a.data_ptr() + 4 * shift, b.data_ptr() + 4 * shift, w)
        for a, b, w in zip(ins, outs, WIDTHS)))
    L.check(lib.gb_densify_apply(ctypes.byref(raw(src, P)), work.data_ptr(), noise.data_ptr(), 0.5,
                                 ctypes.byref(opts), ctypes.byref(raw(out, n_new)), states,
                                 len(WIDTHS), stream), "apply")
    torch.cuda.synchronize()
    for f, t in src.items():
        np.testing.assert_array_equal(out[f].cpu().numpy(), t.cpu().numpy()[parent], err_msg=f)
    for a, b, w in zip(ins, outs, WIDTHS):
        rows = a.cpu().numpy()[shift:].reshape(P, w)[parent]
        rows[new] = 0.0
        got = b.cpu().numpy()
        np.testing.assert_array_equal(got[shift:shift + n_new * w].reshape(n_new, w), rows)
        assert np.all(got[:shift] == -7.0) and np.all(got[shift + n_new * w:] == -7.0)
