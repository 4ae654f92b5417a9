"""Adam over several arrays in one launch equals one call per array, bit for bit: empty arrays,
sizes around a thread's four values and a workgroup's, and more arrays than a launch takes."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1,), (3, 0, 4), (5, 1023, 1024, 1025, 2),
                                   (7, 0, 1, 2, 3, 4, 5, 0, 6, 4097, 300001)])
def test_adam_groups_equal_single_calls(sizes):
    from paper_2412_12734_amd import _lib as L
    lib = L.load()
    rng = np.random.default_rng(len(sizes))
    dev = lambda n: torch.from_numpy(rng.standard_normal(n).astype(np.float32)).cuda()
    a = [[dev(max(n, 1)) for _ in range(3)] + [dev(max(n, 1)).abs()] for n in sizes]
    b = [[t.clone() for t in row] for row in a]
    bits = [[torch.zeros(max(n, 1), dtype=torch.int16, device="cuda") for n in sizes]
            for _ in range(2)]
    lrs = [float(np.float32(10.0 ** -(1 + k % 4))) for k in range(len(sizes))]
    copy = lambda side, k: bits[side][k].data_ptr() if k % 2 == 0 else None
    stream = torch.cuda.current_stream().cuda_stream
    for step in (1, 2):
        groups = (L.GbAdamGroup * len(sizes))(*(
            L.GbAdamGroup(n, p.data_ptr(), g.data_ptr(), m.data_ptr(), v.data_ptr(), copy(0, k),
                          lrs[k]) for k, (n, (p, g, m, v)) in enumerate(zip(sizes, a))))
        assert lib.gb_adam_steps(groups, len(sizes), step, 0.9, 0.999, 1e-15, stream) == L.GB_OK
        for k, (n, (p, g, m, v)) in enumerate(zip(sizes, b)):
            assert lib.gb_adam_step(n, p.data_ptr(), g.data_ptr(), m.data_ptr(), v.data_ptr(),
                                    step, lrs[k], 0.9, 0.999, 1e-15, copy(1, k),
                                    stream) == L.GB_OK
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        for s, t in zip(x, y):
            assert torch.equal(s, t)
    for s, t in zip(*bits):
        assert torch.equal(s, t)
    # one bad array: nothing is updated
    before = a[0][0].clone()
    groups = (L.GbAdamGroup * 2)(
        L.GbAdamGroup(sizes[0], *(t.data_ptr() for t in a[0]), None, 0.1),
        L.GbAdamGroup(4, None, None, None, None, None, 0.1))
    assert lib.gb_adam_steps(groups, 2, 3, 0.9, 0.999, 1e-15, stream) == L.GB_ERR_ARG
    torch.cuda.synchronize()
    assert torch.equal(before, a[0][0])
