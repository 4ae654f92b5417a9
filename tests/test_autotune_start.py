"""The autotuner starts from what the library does when nothing is chosen: batch sizes of 0 (chosen by
grid side and number of tiles, with values that no explicit size gives) are measured first and are
among the candidates, so that tuned options cannot lose to untuned ones."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2412_12734_amd import autotune as at
from paper_2412_12734_amd.render import Options


def tune(N, cost, base=None):
    splats = types.SimpleNamespace(P=100, N=N, textures=torch.zeros(1))
    return at.autotune(splats, [types.SimpleNamespace(width=64, height=48)], base=base, cost=cost)


@pytest.mark.parametrize("N", [1, 2, 4, 8])
def test_the_librarys_own_batches_are_measured_first_and_can_win(N):
    seen = []

    def cost(o):
        seen.append((o.batch, o.batch_bwd))
        return 1.0 + (o.batch != 0) + (o.batch_bwd != 0)

    best, rec = tune(N, cost)
    assert seen[0] == (0, 0)
    assert (best.batch, best.batch_bwd) == (0, 0) and rec["ms"] == rec["default_ms"] == 1.0
    assert {8, 16, 32, 64} <= {b for b, _ in seen} and {8, 16, 32} <= {b for _, b in seen}


def test_a_given_batch_is_the_start_and_zero_a_candidate():
    seen = []

    def cost(o):
        seen.append((o.batch, o.batch_bwd))
        return 1.0 + (o.batch != 0) + (o.batch_bwd != 8)

    best, _ = tune(8, cost, Options(batch=32, batch_bwd=8))
    assert seen[0] == (32, 8) and (best.batch, best.batch_bwd) == (0, 8)


def test_a_better_explicit_batch_is_found_from_zero():
    best, _ = tune(4, lambda o: abs(o.batch - 32) + abs(o.batch_bwd - 16))
    assert (best.batch, best.batch_bwd) == (32, 16)
