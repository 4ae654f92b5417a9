"""CPU emulation of how the blends cut a tile's list into passes (pass_size), in 32-bit unsigned
arithmetic: lists that end at the last pair slot there can be, 2^32 - 16, are walked once and to
their end, as those at the front are."""
import pytest

M = 1 << 32


def pass_size(b, end, most):
    return min((end - b) % M, most)


def forward(start, end):
    seen, b, n, loads = [], start, 0, []
    loads.append([(start + lane) % M for lane in range(64) if lane < pass_size(start, end, 64)])
    while b < end:
        n = pass_size(b, end, 64)
        seen.append([(b + lane) % M for lane in range(64) if lane < n])
        loads.append([(b + n + lane) % M for lane in range(64)
                      if lane < pass_size((b + n) % M, end, 64)])
        b = (b + n) % M
        assert len(seen) <= 10
    assert loads[:len(seen)] == seen and loads[len(seen):] in ([], [[]])
    return [e for p in seen for e in p]


def backward(start, last, most):
    seen, pend = [], last
    while pend > start:
        n = pass_size(start, pend, most)
        base = (pend - n) % M
        seen += reversed([(base + lane) % M for lane in range(64) if lane < n])
        pend = base
        assert len(seen) <= 600
    return seen


@pytest.mark.parametrize("count", [0, 1, 31, 32, 33, 47, 48, 49, 63, 64, 65, 130])
@pytest.mark.parametrize("end", [300, M - 16])
def test_every_entry_once(end, count):
    want = list(range(end - count, end))
    assert forward(end - count, end) == want
    for most in (32, 48, 64):
        assert backward(end - count, end, most) == want[::-1]
