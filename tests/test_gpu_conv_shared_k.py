"""fp32 layers of small images: eight waves share a tile's K sum; a batch too
large for that adds the same parts in turn. Each image of a batch equals its
own launch bit for bit, and both stay within fp32 accumulation of the oracle."""
import numpy as np
import pytest
import torch

from oracle import vinet as O

pytestmark = pytest.mark.gpu


# (n of the batch, cin, cout, h, w, stride, transposed)
@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", [
    (60, 64, 64, 11, 13, 1, False),    # two parts; 64 x 64 in the batch
    (80, 40, 33, 9, 7, 1, False),      # second slice mostly padding, odd output channels
    (40, 256, 256, 8, 17, 1, False),   # eight parts; 64 x 128 in the batch
    (9, 256, 128, 15, 33, 2, False),   # stride 2
    (20, 96, 20, 33, 31, 2, False),    # three parts, 128 x 32 in the batch
    (6, 384, 72, 12, 20, 1, False),    # twelve slices in six parts
    (12, 512, 128, 8, 9, 0, True),     # sixteen slices in eight parts, one phase per workgroup
    (30, 128, 5, 20, 31, 0, True),     # phase-merged, 20 columns
    (30, 64, 16, 19, 23, 0, True),     # phase-merged, 64 columns
])
def test_batch_equals_single_and_oracle(n, cin, cout, h, w, stride, transposed):
    from paper_2112_10603_amd import op_conv
    print(f"case shared K n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed}", flush=True)
    rng = np.random.default_rng(cin + cout + h)
    x = rng.standard_normal((n, cin, h, w)).astype(np.float32)
    shape = (cin, cout, 4, 4) if transposed else (cout, cin, 3, 3)
    wt = (rng.standard_normal(shape) / np.sqrt(cin * (4 if transposed else 9))).astype(np.float32)
    b = rng.standard_normal(cout).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    got = op_conv(xd, wt, b, **kw)
    for i in (0, n // 2, n - 1):
        one = op_conv(xd[i:i + 1].contiguous(), wt, b, **kw)
        assert torch.equal(got[i:i + 1], one)
        assert torch.equal(one, op_conv(xd[i:i + 1].contiguous(), wt, b, noalloc=True, **kw))
    xi, w64, b64 = x[n - 1].astype(np.float64), wt.astype(np.float64), b.astype(np.float64)
    conv = (lambda q, v, c: O.conv_transpose2d(q, v, c)) if transposed else (lambda q, v, c: O.conv2d(q, v, c, stride))
    ref, absref = conv(xi, w64, b64), conv(np.abs(xi), np.abs(w64), np.abs(b64))
    err = np.abs(got[n - 1].cpu().numpy().astype(np.float64) - ref)
    # fp32 accumulation over K terms, as for the other tiles
    assert np.all(err <= 2e-5 * absref + 1e-6)
