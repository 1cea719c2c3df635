"""The operator's default tile is the network's: the direct-weight kernel at
sizes past the no-allocation scratch too (an fp32 image then equals itself in
any batch), and elsewhere the tile rule, whose every choice gives the bits of
an explicit tile."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _data(n, cin, cout, h, w, transposed, seed):
    rng = np.random.default_rng(seed)
    x = torch.rand((n, cin, h, w), generator=torch.Generator().manual_seed(seed)).cuda()
    shape = (cin, cout, 4, 4) if transposed else (cout, cin, 3, 3)
    wt = (rng.standard_normal(shape) / np.sqrt(cin * (4 if transposed else 9))).astype(np.float32)
    return x, wt, rng.standard_normal(cout).astype(np.float32)


@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", [
    (9, 64, 64, 128, 128, 1, False),
    (12, 128, 64, 64, 120, 0, True),
    (16, 256, 256, 60, 64, 2, False),
])
def test_fp32_image_does_not_depend_on_its_batch(n, cin, cout, h, w, stride, transposed):
    from paper_2112_10603_amd import op_conv
    print(f"case op default n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed}", flush=True)
    x, wt, b = _data(n, cin, cout, h, w, transposed, 7)
    assert x.nbytes + n * cout * h * w * 4 > 64 << 20  # past the scratch of the no-allocation entry point
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    got = op_conv(x, wt, b, **kw)
    for i in (0, n - 1):
        one = op_conv(x[i:i + 1].contiguous(), wt, b, **kw)
        assert torch.equal(got[i:i + 1], one)
        assert torch.equal(one, op_conv(x[i:i + 1].contiguous(), wt, b, noalloc=True, **kw))


def test_fp32_large_image():
    """64 -> 64 at 540 x 960 (unet.enc4 of a 4K view) on 128 x 64 direct tiles."""
    from paper_2112_10603_amd import op_conv
    print("case op default 64 -> 64 at 540x960", flush=True)
    x, wt, b = _data(1, 64, 64, 540, 960, False, 9)
    got = op_conv(x, wt, b, precision="fp32")
    plain = op_conv(x, wt, b, precision="fp32", n_tile=64)
    terms = op_conv(x, np.abs(wt), np.abs(b), precision="fp32", n_tile=64)
    assert not torch.equal(got, plain)  # the direct kernel sums in another order
    # two fp32 accumulations over K terms, as for the other tiles
    assert torch.all((got - plain).abs() <= 4e-5 * terms + 1e-6)


@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", [
    (2, 64, 256, 136, 136, 1, False),    # two-group halo tile
    (2, 64, 128, 136, 136, 1, False),    # 128-column halo tile
    (2, 64, 64, 136, 136, 1, False),     # resident weights, 64 columns
    (2, 64, 32, 136, 136, 1, False),     # 32 columns
    (2, 512, 8, 136, 136, 1, False),     # halo kernel: the weights fit no LDS
    (1, 256, 64, 240, 240, 0, True),     # four phases per halo tile
    (2, 256, 128, 136, 136, 0, True),    # two phases
    (3, 128, 5, 136, 137, 0, True),      # phase-merged
    (1, 18, 128, 33, 47, 2, False),      # few-channel kernel, 128 columns
    (1, 18, 64, 33, 47, 2, False),
    (2, 16, 32, 19, 65, 1, False),
    (1, 18, 20, 33, 47, 2, False),       # no 16-byte runs of output channels: the generic tile
    (1, 40, 256, 64, 64, 2, False),      # 64 columns while they are one round of workgroups
    (4, 40, 256, 150, 150, 2, False),    # 128 columns
    (12, 40, 256, 150, 150, 2, False),   # 256 columns
])
@pytest.mark.parametrize("act_out", [False, True])
def test_bf16_default_equals_explicit_tile(n, cin, cout, h, w, stride, transposed, act_out):
    from paper_2112_10603_amd import op_conv
    print(f"case op default bf16 n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed} {act_out}", flush=True)
    x, wt, b = _data(n, cin, cout, h, w, transposed, cin + cout)
    kw = dict(stride=max(stride, 1), transposed=transposed, relu=True, precision="bf16", act_out=act_out)
    assert torch.equal(op_conv(x, wt, b, **kw), op_conv(x, wt, b, n_tile=32, **kw))
