"""fp32 layers that meet infinities and NaN: an image's outputs do not depend
on its batch, finite outputs beside a non-finite one keep their values, and
such inputs do not cost orders of magnitude more time."""
import numpy as np
import pytest
import torch

from oracle import vinet as O
from synth.weights import make_weights, save_ffvw

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


# (n of the batch, cin, cout, h, w, stride, transposed): another tile alone than in the batch
@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", [
    (8, 32, 256, 45, 80, 1, False),    # 64 x 64 against 128 x 128
    (40, 32, 64, 21, 37, 1, False),    # 64 x 64 against 128 x 64
    (60, 64, 64, 11, 13, 1, False),    # shared K against 64 x 64
    (40, 256, 256, 8, 17, 1, False),   # shared K against 64 x 128
    (9, 256, 128, 15, 33, 2, False),
    (20, 96, 20, 33, 31, 2, False),    # shared K against 128 x 32
    (12, 512, 128, 8, 9, 0, True),
    (30, 128, 5, 20, 31, 0, True),
])
def test_batch_equals_single(n, cin, cout, h, w, stride, transposed):
    from paper_2112_10603_amd import op_conv
    print(f"case nonfinite n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed}", flush=True)
    rng = np.random.default_rng(cin + cout + h)
    x = rng.standard_normal((n, cin, h, w)).astype(np.float32)
    shape = (cin, cout, 4, 4) if transposed else (cout, cin, 3, 3)
    wt = (rng.standard_normal(shape) / np.sqrt(cin * (4 if transposed else 9))).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    clean = x[0].copy()
    x[0, 3, 2, 3] = np.inf
    x[0, 7, h - 1, w // 2] = -np.inf
    x[0, 1, h // 2, w - 1] = np.nan
    x[0, 5, h // 2, 1] = 3.4e38
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    one = op_conv(xd[:1].contiguous(), wt, b, **kw).cpu().numpy()
    np.testing.assert_array_equal(op_conv(xd, wt, b, **kw).cpu().numpy()[:1], one)
    ref = op_conv(xd[:1].contiguous(), wt, b, n_tile=32, **kw).cpu().numpy()
    np.testing.assert_array_equal(np.isnan(one), np.isnan(ref))
    np.testing.assert_array_equal(np.isposinf(one), np.isposinf(ref))
    np.testing.assert_array_equal(np.isneginf(one), np.isneginf(ref))
    # outputs that read none of the planted values: those of the clean image
    plain = op_conv(torch.from_numpy(clean[None]).cuda(), wt, b, **kw).cpu().numpy()
    planted = ~np.isfinite(x[0]).all(0) | (np.abs(x[0]) > 1e38).any(0)
    near = np.pad(planted, 1)
    near = sum(near[dy:dy + h, dx:dx + w].astype(int) for dy in range(3) for dx in range(3)) > 0
    # (a phase-merged transposed conv reads the whole 3 x 3 neighbourhood, with zero weights)
    near = near.repeat(2, 0).repeat(2, 1) if transposed else near[::stride, ::stride]
    far = np.broadcast_to(~near, one.shape)
    assert far.any()
    np.testing.assert_array_equal(one[far], plain[far])
    fin = np.isfinite(ref)
    x64, w64, b64 = x[0].astype(np.float64), wt.astype(np.float64), b.astype(np.float64)
    x64 = np.where(np.isfinite(x64), x64, 0)
    conv = O.conv_transpose2d if transposed else (lambda p, q, r: O.conv2d(p, q, r, stride))
    want, terms = conv(x64, w64, b64), conv(np.abs(x64), np.abs(w64), np.abs(b64))
    # fp32 accumulation over K terms
    assert np.all((np.abs(one[0] - want) <= 2e-5 * terms + 1e-6)[fin[0]])


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
