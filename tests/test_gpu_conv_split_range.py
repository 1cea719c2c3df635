"""fp32 convolutions at the ends of the float range. Layers whose weights the
three-way bf16 split cannot hold (near the largest float, infinite, NaN) give
what the fp32 matrix instruction gives; tiny weights and activations keep
their precision."""
import numpy as np
import pytest
import torch

from oracle import vinet as O

pytestmark = pytest.mark.gpu

LAYERS = [(1, False, 64), (2, False, 128), (0, True, 32), (0, True, 5)]  # (stride, transposed, cout)


def _data(cout, transposed, seed, cin=64, h=24, w=20):
    rng = np.random.default_rng(seed)
    x = np.maximum(rng.standard_normal((1, cin, h, w)), 0).astype(np.float32)
    shape = (cin, cout, 4, 4) if transposed else (cout, cin, 3, 3)
    wt = (rng.standard_normal(shape) / np.sqrt(cin * (4 if transposed else 9))).astype(np.float32)
    return x, wt, rng.standard_normal(cout).astype(np.float32)


@pytest.mark.parametrize("stride,transposed,cout", LAYERS)
@pytest.mark.parametrize("value", [3.4e38, -3.3962e38, 2.0 ** 110, np.inf, -np.inf, np.nan])
def test_extreme_weights(stride, transposed, cout, value):
    from paper_2112_10603_amd import op_conv
    print(f"case fp32 weight {value} s={stride} T={transposed} cout={cout}", flush=True)
    x, wt, b = _data(cout, transposed, 5)
    x *= 0.25  # one extreme weight leaves the sums finite
    wt[1, 2, 1, 1] = value
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    ref = op_conv(xd, wt, b, n_tile=32, **kw).cpu().numpy()
    for noalloc in (False, True):
        got = op_conv(xd, wt, b, noalloc=noalloc, **kw).cpu().numpy()
        np.testing.assert_array_equal(got, ref)
    if np.isfinite(value):
        x64, w64, b64 = (v.astype(np.float64) for v in (x[0], wt, b))
        conv = O.conv_transpose2d if transposed else (lambda p, q, r: O.conv2d(p, q, r, stride))
        want, terms = conv(x64, w64, b64), conv(np.abs(x64), np.abs(w64), np.abs(b64))
        # fp32 accumulation over K terms; sums past the largest float are infinite
        fits = terms < 3.4e38
        assert fits.any()
        assert np.all(np.abs(ref[0].astype(np.float64) - want)[fits] <= (2e-5 * terms + 1e-6)[fits])


@pytest.mark.parametrize("stride,transposed,cout", LAYERS)
@pytest.mark.parametrize("xs,ws", [(1e-30, 1.0), (1e-36, 1.0), (2e-37, 2.0 ** 60), (1.0, 1e-36), (2.0 ** 60, 2e-37),
                                   (1e-17, 1e-18)])
def test_tiny_values(stride, transposed, cout, xs, ws):
    """No further from float64 than the fp32 matrix instruction (5 % for the
    spread of a sample, as for ordinary magnitudes), and within fp32
    accumulation over K terms of it."""
    from paper_2112_10603_amd import op_conv
    print(f"case fp32 tiny x {xs} w {ws} s={stride} T={transposed} cout={cout}", flush=True)
    x, wt, b = _data(cout, transposed, 11)
    x, wt, b = x * np.float32(xs), wt * np.float32(ws), np.zeros_like(b)
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    got = op_conv(xd, wt, b, **kw).cpu().numpy()[0].astype(np.float64)
    plain = op_conv(xd, wt, b, n_tile=32, **kw).cpu().numpy()[0].astype(np.float64)
    x64, w64, b64 = (v.astype(np.float64) for v in (x[0], wt, b))
    conv = O.conv_transpose2d if transposed else (lambda p, q, r: O.conv2d(p, q, r, stride))
    want, terms = conv(x64, w64, b64), conv(np.abs(x64), np.abs(w64), np.abs(b64))
    e_got, e_plain = np.linalg.norm(got - want), np.linalg.norm(plain - want)
    print(f"  error {e_got / np.linalg.norm(want):.2e} fp32 MFMA {e_plain / np.linalg.norm(want):.2e}")
    assert e_got <= 1.05 * e_plain
    assert np.all(np.abs(got - want) <= 2e-5 * terms)


def test_net_with_extreme_weights(tmp_path):
    """Layers of both kinds in one fp32 net, alone and in a batch."""
    from paper_2112_10603_amd import Net
    from synth import scenes
    from synth.weights import make_weights, save_ffvw
    print("case fp32 net with extreme weights", flush=True)
    W = make_weights(0)
    for name in ("vib1.conv4", "vib2.convT1", "unet.enc3", "ctx.conv2"):
        W[name][0][0, 1, 1, 1] = 2.0 ** 110
    path = str(tmp_path / "w.ffvw")
    save_ffvw(path, W, 32, True, 0)
    dev = torch.device("cuda:0")
    arc = scenes.camera_arc(3, 48, 80, 2, 64, (3.0, 8.0), 4.0, 0.01).to(dev)
    pair, ts = (arc[0].contiguous(), arc[1].contiguous()), [0.2, 0.5, 0.8]
    net = Net(path, "fp32", 0)
    batch = net.interpolate([pair], ts)[0].cpu().numpy()
    for k, t in enumerate(ts):
        np.testing.assert_array_equal(net.interpolate([pair], [t])[0, 0].cpu().numpy(), batch[k])
    net.close()
