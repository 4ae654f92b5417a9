"""What Trainer.step hands to the loss as the target image: a buffer of the batch's pixels, or with
one view the image itself where it has every pixel. An image of too few rows is refused (the loss
reads as many values as were rendered), whichever way it would go. On the CPU, with the library's
calls replaced."""
import types

import pytest
import torch

from paper_2412_12734_amd import train as T

W, H = 6, 4
N_PX = W * H


def step_target(targets, batch=(0,)):
    """The tensor that the loss of one step is called with, and its values then."""
    seen = []
    state = types.SimpleNamespace(device="cpu", activate=lambda: types.SimpleNamespace(n_texels=0),
                                  backward_activations=lambda g: g, adam=lambda g: None)
    tr = T.Trainer(state, [types.SimpleNamespace(width=W, height=H)] * 2, targets)
    tr.rast = types.SimpleNamespace(set_views=lambda v: None,
                                    forward=lambda sp, rgb, t, zero_grads: (rgb, t),
                                    backward=lambda *a: {})
    tr.loss_fn = lambda rgb, target, scale, loss, d_rgb: seen.append((rgb, target))
    tr.step(list(batch))
    (rgb, target), = seen
    assert rgb.shape == (len(batch) * N_PX, 3)
    assert target.shape == rgb.shape and target.dtype == torch.float32 and target.is_contiguous()
    return target


@pytest.mark.parametrize("rows", [0, 2, N_PX - 1])
@pytest.mark.parametrize("batch", [(0,), (0, 1)])
def test_image_of_too_few_rows_is_refused(rows, batch):
    with pytest.raises(RuntimeError):
        step_target(torch.rand(2, rows, 3), batch)


@pytest.mark.parametrize("batch", [(0,), (1, 0)])
def test_image_of_one_row_is_one_colour(batch):
    targets = torch.rand(2, 1, 3)
    got = step_target(targets, batch).view(len(batch), N_PX, 3)
    assert torch.equal(got, targets[list(batch)].expand(-1, N_PX, -1))


@pytest.mark.parametrize("rows", [N_PX, N_PX + 5])
def test_whole_image_is_compared_where_it_lies(rows):
    targets = torch.rand(2, rows, 3)
    got = step_target(targets, (1,))
    assert torch.equal(got, targets[1, :N_PX])
    if targets[1].data_ptr() % 16 == 0:
        assert got.data_ptr() == targets[1].data_ptr()


@pytest.mark.parametrize("make", [
    lambda t: t.double(), lambda t: t.to(torch.bfloat16),
    lambda t: torch.cat([torch.zeros(1), t.reshape(-1)])[1:].view(t.shape),  # misaligned
], ids=["float64", "bfloat16", "misaligned"])
def test_other_images_are_copied(make):
    targets = make(torch.rand(2, N_PX, 3))
    for batch in ((1,), (0, 1)):
        got = step_target(targets, batch)
        assert torch.equal(got, targets[list(batch)].float().reshape(-1, 3))
        assert got.data_ptr() % 16 == 0 and got.data_ptr() != targets[batch[0]].data_ptr()
