"""The band sums of the Eq. 3 loss on values whose float32 sums lose the small
ones: rows of alternating sign along x have no coarser levels (the binomial
filter's response at the Nyquist frequency is 0), so the loss is the mean
magnitude, exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w", [(64, 256), (128, 128), (66, 640)])
@pytest.mark.parametrize("rows", [(1.0, 2.0 ** -23), (2.0 ** -23, 1.0)])
def test_band_sum_keeps_small_values(h, w, rows):
    from paper_2112_10603_amd import lap_loss
    print(f"case lap sum {h}x{w} rows {rows}", flush=True)
    x = np.zeros((1, 3, h, w), np.float32)
    for k in range(2):
        x[:, :, k::2, 0::2] = rows[k]
        x[:, :, k::2, 1::2] = -rows[k]
    xd = torch.from_numpy(x).cuda()
    loss, grad = lap_loss(xd, torch.zeros_like(xd), grad=True)
    # (1 + 2^-23) / 2 is a float32
    assert loss.item() == (1.0 + 2.0 ** -23) / 2
    assert lap_loss(xd, torch.zeros_like(xd)).item() == loss.item()
    assert torch.isfinite(grad).all()
