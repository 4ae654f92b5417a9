"""CPU emulation of the backward's row sums by masked DPP adds: which lane ends with which value,
that the owner lanes of a row hold each value's row total exactly once (a value in two parts
adds up from both), and that the ordered variant adds a wave's lanes in its stated order, to the
bit, for either direction of the hardware swap."""
import numpy as np
import pytest


def mirror(v):
    return v.reshape(-1, 16)[:, ::-1].reshape(-1)


def half_mirror(v):
    return v.reshape(-1, 8)[:, ::-1].reshape(-1)


def quad(v, perm):
    return v.reshape(-1, 4)[:, perm].reshape(-1)


LANE = np.arange(64)
B3, B2, B1, B0 = (LANE >> k & 1 == 1 for k in (3, 2, 1, 0))


def pair(a, b, move, mask):
    """a + moved a in every lane, then b + moved b in the masked lanes."""
    return np.where(mask, b + move(b), a + move(a))


def row_sums(v):
    K = len(v)
    q2, q1 = (lambda x: quad(x, [2, 3, 0, 1])), (lambda x: quad(x, [1, 0, 3, 2]))
    if K == 3:
        x = pair(pair(v[0], v[1], mirror, B3), v[2], half_mirror, B2)
        x = x + q2(x)
        return x + q1(x)
    t = [pair(v[2 * i], v[2 * i + 1], mirror, B3) for i in range(K // 2)]
    if K == 6:
        s, z = pair(t[0], t[1], half_mirror, B2), t[2]
        x = np.where(B1, z, s) + q2(np.where(B1, s, z))
        return x + q1(x)
    s = [pair(t[2 * i], t[2 * i + 1], half_mirror, B2) for i in range(3)]
    x = np.where(B1, s[1], s[0]) + q2(np.where(B1, s[0], s[1]))
    y = s[2] + q2(s[2])
    return np.where(B0, y, x) + q1(np.where(B0, x, y))


def row_slot(K, l):
    b3, b2, b1, b0 = l >> 3 & 1, l >> 2 & 1, l >> 1 & 1, l & 1
    if K == 12:
        return (-1 if b1 else 8 + 2 * b2 + b3) if b0 else 4 * b1 + 2 * b2 + b3
    if K == 6:
        return -1 if b0 else 2 * (2 if b1 else b2) + b3
    return -1 if b1 or b0 else (2 if b2 else b3)


@pytest.mark.parametrize("K", [3, 6, 12])
def test_owner_lanes_hold_each_row_total_once(K):
    v = np.random.default_rng(K).standard_normal((K, 64))
    got, out = np.zeros((4, K)), row_sums(v)
    for l in range(64):
        if row_slot(K, l & 15) >= 0:
            got[l // 16, row_slot(K, l & 15)] += out[l]
    np.testing.assert_allclose(got, v.reshape(K, 4, 16).sum(2).T, atol=1e-13)


def swap(a, b, group, upper):
    """One swap step: lanes of one side end with a summed over the lane pair, the other with b."""
    side = ((LANE & group) != 0) == upper
    return np.where(side, b + b[LANE ^ group], a + a[LANE ^ group]).astype(np.float32), side


@pytest.mark.parametrize("upper", [False, True])
def test_ordered_sums_add_in_the_stated_order(upper):
    v = np.random.default_rng(5).standard_normal((12, 64)).astype(np.float32)
    a = [swap(v[2 * i], v[2 * i + 1], 32, upper) for i in range(6)]
    h = a[0][1]
    b = [swap(a[2 * i][0], a[2 * i + 1][0], 16, upper) for i in range(3)]
    r = b[0][1]
    x = pair(b[0][0], b[1][0], mirror, B3)
    x = pair(x, b[2][0] + mirror(b[2][0]), half_mirror, B2)
    x = x + quad(x, [3, 2, 1, 0])
    x = x + quad(x, [1, 0, 3, 2])
    assert x.dtype == np.float32
    seen = []
    for l in range(64):
        if not 0x0111 >> (l & 15) & 1:
            continue
        k = 4 * (2 if l & 4 else l >> 3 & 1) + 2 * int(r[l]) + int(h[l])
        want = v[k]
        for m in (32, 16, 15, 7, 3, 1):
            want = want + want[LANE ^ m]
        assert x[l] == want[l]
        seen.append(k)
    assert sorted(seen) == list(range(12))
