"""The bf16 output head, which walks down strips of 32 pixels two rows a
step: its output against the head computed in float64 from the activations
and the blend that it read, at sizes around a strip, for both channel counts
of the matrix-core kernel."""
import numpy as np
import pytest
import torch

from oracle import vinet as O
from synth import scenes
from synth.weights import write_weights_file

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("base_width", [32, 64])
@pytest.mark.parametrize("H,W", [(2, 2), (15, 31), (16, 32), (17, 33), (48, 64), (61, 259), (300, 97)])
def test_head_strips(tmp_path, base_width, H, W):
    from paper_2112_10603_amd import Net
    print(f"case head strips {H}x{W} base {base_width}", flush=True)
    wfile = write_weights_file(str(tmp_path / "w.ffvw"), seed=2, base_width=base_width)
    arc = scenes.camera_arc(H + W, max(H, 16), max(W, 16), 2, 64, (1.0, 4.0), 4.0, 0.01)
    xl, xr = (arc[i, :, :H, :W].contiguous().to(DEV) for i in range(2))
    net = Net(wfile, "bf16", 0)
    net.set_debug(True)
    out = net.interpolate([(xl, xr)], [0.5])[0, 0].cpu().numpy().astype(np.float64)
    u4, I2 = (net.debug_tap(n).cpu().numpy().astype(np.float64) for n in ("u4", "I2"))
    net.close()
    _, _, w, b = O.load_weights(wfile)["layers"]["unet.head"]
    w = torch.from_numpy(w).float().bfloat16().double().numpy()  # as every bf16 layer's
    z = O.conv2d(u4, w, b, 1)[:, :H, :W]
    terms = O.conv2d(np.abs(u4), np.abs(w), np.abs(b), 1)[:, :H, :W]
    ref = np.clip(I2[:3, :H, :W] + 2.0 / (1.0 + np.exp(-z)) - 1.0, 0.0, 1.0)
    # z: up to 289 terms summed in fp32, each step off by 2^-24 of the sum at
    # most; the sigmoid's slope is 1/4, doubled; a few roundings of the rest
    tol = 0.5 * 289 * 2.0 ** -24 * terms + 2e-6
    assert np.all(np.abs(out - ref) <= tol)
