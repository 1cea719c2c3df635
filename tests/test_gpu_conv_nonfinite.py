"""fp32 layers that meet values their operands' split cannot hold: such inputs
do not cost orders of magnitude more time."""
import numpy as np
import pytest
import torch

from synth.weights import make_weights, save_ffvw

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _time(net, pair, n=5):
    net.interpolate([pair], [0.5])
    ms = []
    for _ in range(n):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        a.record()
        net.interpolate([pair], [0.5])
        torch.cuda.synchronize()
        b.record()
        torch.cuda.synchronize()
        ms.append(a.elapsed_time(b))
    return min(ms)


@pytest.mark.parametrize("value", [1e36, np.inf])
def test_unsplittable_image_time(tmp_path, value):
    """A view of an image whose every pixel is past the split's range (the
    weights are positive and their sums 0.9: 1e36 keeps its magnitude through
    every layer, infinities last through the first stage and ContextNet). A
    wave that meets such values redoes its tile with fp32 matrix
    instructions, 16 / 6 of the time of the six products, and reads its
    operands from global memory itself, a few times slower than from LDS: 12
    times an ordinary view's time is never reached."""
    from paper_2112_10603_amd import Net
    print(f"case unsplittable image time {value}", flush=True)
    path = str(tmp_path / "w.ffvw")
    W = {}
    for name, (w, b) in make_weights(0).items():
        transposed = "convT" in name or "dec" in name
        gain = np.abs(w).sum((0, 2, 3) if transposed else (1, 2, 3)).max() / (4 if transposed else 1)
        W[name] = ((np.abs(w) * (0.9 / gain)).astype(np.float32), np.abs(b))
    save_ffvw(path, W, 32, True, 0)
    net = Net(path, "fp32", 0)
    g = torch.Generator().manual_seed(3)
    xl, xr = (torch.rand((3, 192, 256), generator=g).to(DEV) for _ in range(2))
    ordinary = _time(net, (xl, xr))
    large = _time(net, (torch.full_like(xl, value), torch.full_like(xl, value)))
    net.close()
    print(f"  ordinary {ordinary:.3f} ms, unsplittable {large:.3f} ms", flush=True)
    assert large <= 12 * ordinary
