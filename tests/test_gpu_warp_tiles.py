"""The warping passes' 64 x 4 tiles: sizes around a tile and a column of
tiles against the oracle, and a batch past the pixel count at which the order
of the tiles changes equal to its views computed alone."""
import numpy as np
import pytest
import torch

from oracle import vinet as O
from synth import scenes
from synth.weights import write_weights_file

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def wfile(tmp_path_factory):
    return write_weights_file(str(tmp_path_factory.mktemp("w") / "w0.ffvw"), seed=0)


@pytest.mark.parametrize("H,W", [(16, 64), (33, 65), (49, 127), (64, 272)])
def test_tile_edges_fp32(wfile, H, W):
    from paper_2112_10603_amd import Net
    print(f"case warp tiles {H}x{W}", flush=True)
    arc = scenes.camera_arc(H + W, H, W, 2, 96, (3.0, 10.0), 6.0, 0.01)
    net = Net(wfile, "fp32", 0)
    got = net.interpolate([(arc[0].to(DEV), arc[1].to(DEV))], [0.5])[0, 0].cpu().numpy()
    net.close()
    ref = O.vinet_forward(arc[0].numpy(), arc[1].numpy(), 0.5, O.load_weights(wfile))
    assert np.abs(got - ref).max() <= 1e-4  # the network's fp32 bound


def test_order_of_large_batch(wfile):
    from paper_2112_10603_amd import Net
    H, W, n_t = 552, 1400, 12  # 24 views of 560 x 1408: 18.9 M pixels
    print(f"case warp tiles batch {H}x{W} x {2 * n_t}", flush=True)
    arc = scenes.camera_arc(5, H, W, 3, 256, (3.0, 10.0), 6.0, 0.01).to(DEV)
    pairs, ts = [(arc[0], arc[1]), (arc[1], arc[2])], [(k + 1) / (n_t + 1) for k in range(n_t)]
    net = Net(wfile, "bf16", 0)
    out = net.interpolate(pairs, ts)
    for p, k in ((0, 0), (1, 5), (1, n_t - 1)):
        assert torch.equal(net.interpolate([pairs[p]], [ts[k]])[0, 0], out[p, k]), (p, k)
    net.close()
