"""The direct-weight conv kernel, which the default tile choice takes for
small grids and for every fp32 layer: bf16 equal bit for bit to an explicit
tile of the implicit-GEMM kernel, fp32 (three-way bf16 split) against the
oracle and no further from it than the fp32 matrix instruction, at every
tile, remainder and slice-ring edge."""
import numpy as np
import pytest
import torch

from oracle import vinet as O

pytestmark = pytest.mark.gpu

# (n, cin, cout, h, w, stride, transposed)
CASES = [
    (1, 64, 64, 5, 7, 1, False),       # one 64 x 64 tile, mostly padding
    (2, 256, 256, 8, 8, 1, False),     # whole tiles
    (1, 64, 33, 17, 9, 1, False),      # odd output channels: no 16-byte runs
    (1, 64, 40, 15, 33, 1, False),
    (1, 128, 256, 33, 47, 2, False),   # stride 2, odd sizes
    (1, 256, 256, 40, 52, 2, False),   # four slices in three halo buffers
    (2, 256, 128, 9, 13, 0, True),     # transposed, one phase per workgroup
    (1, 512, 128, 45, 80, 0, True),    # 128 x 64 tiles, eight slices in six buffers
    (3, 128, 5, 20, 31, 0, True),      # phase-merged, 20 columns
    (1, 64, 16, 19, 23, 0, True),      # phase-merged, 64 columns
    (1, 64, 256, 68, 60, 1, False),    # 128 x 64 tiles
    (1, 64, 256, 68, 120, 1, False),   # 128 x 128 tiles
    (1, 64, 256, 135, 240, 1, False),  # 128 x 256 tiles
    (1, 64, 128, 90, 160, 0, True),    # 256 x 128 tiles
]


def _data(cin, cout, n, h, w, transposed, seed):
    rng = np.random.default_rng(seed)
    x = np.maximum(rng.standard_normal((n, cin, h, w)), 0).astype(np.float32)
    if transposed:
        wt = (rng.standard_normal((cin, cout, 4, 4)) / np.sqrt(4 * cin)).astype(np.float32)
    else:
        wt = (rng.standard_normal((cout, cin, 3, 3)) / np.sqrt(9 * cin)).astype(np.float32)
    return x, wt, rng.standard_normal(cout).astype(np.float32)


def _ref(x, w, b, stride, transposed):
    x, w, b = (v.astype(np.float64) for v in (x, w, b))
    return np.stack([O.conv_transpose2d(i, w, b) if transposed else O.conv2d(i, w, b, stride) for i in x])


@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", CASES)
@pytest.mark.parametrize("act_out", [False, True])
def test_direct_bf16_equals_explicit_tile(n, cin, cout, h, w, stride, transposed, act_out):
    from paper_2112_10603_amd import op_conv
    print(f"case direct bf16 n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed}", flush=True)
    x, wt, b = _data(cin, cout, n, h, w, transposed, cin + cout + h)
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, relu=True, precision="bf16", act_out=act_out)
    got = op_conv(xd, wt, b, **kw)
    assert torch.equal(got, op_conv(xd, wt, b, n_tile=32, **kw))
    assert torch.equal(got, op_conv(xd, wt, b, noalloc=True, **kw))


F32_CASES = CASES[:11] + [
    (2, 3, 16, 17, 23, 2, False),      # slices padded with zero channels
    (1, 18, 128, 12, 20, 2, False),
    (1, 16, 32, 21, 18, 1, False),
    (1, 40, 33, 7, 7, 1, False),       # a whole slice and a quarter
    (1, 24, 7, 4, 3, 0, True),
    (1, 128, 256, 70, 66, 1, False),   # 128 x 128 tiles, remainders both ways
    (1, 256, 128, 24, 36, 0, True),    # 64 x 128 tiles
    (1, 64, 32, 40, 40, 1, False),     # 128 x 32 tiles
]


@pytest.mark.parametrize("n,cin,cout,h,w,stride,transposed", F32_CASES)
def test_direct_f32_vs_oracle(n, cin, cout, h, w, stride, transposed):
    from paper_2112_10603_amd import op_conv
    print(f"case direct fp32 n={n} cin={cin} cout={cout} {h}x{w} s={stride} T={transposed}", flush=True)
    x, wt, b = _data(cin, cout, n, h, w, transposed, cin * 3 + cout + h)
    ref = _ref(x, wt, b, stride, transposed)
    absref = _ref(x, np.abs(wt), np.abs(b), stride, transposed)
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    got = op_conv(xd, wt, b, **kw).cpu().numpy().astype(np.float64)
    # fp32 accumulation over K terms, as for the other tiles
    assert np.all(np.abs(got - ref) <= 2e-5 * absref + 1e-6)
    plain = op_conv(xd, wt, b, n_tile=32, **kw).cpu().numpy().astype(np.float64)
    e_split, e_plain = np.linalg.norm(got - ref), np.linalg.norm(plain - ref)
    print(f"  error split {e_split / np.linalg.norm(ref):.2e} fp32 MFMA {e_plain / np.linalg.norm(ref):.2e}")
    # (both are a few hundred roundings; 5 % for the spread of small samples)
    assert e_split <= 1.05 * e_plain


@pytest.mark.parametrize("stride,transposed,cout", [(1, False, 64), (2, False, 128), (0, True, 32), (0, True, 5)])
def test_direct_f32_extreme_values(stride, transposed, cout):
    """Infinities, NaN and magnitudes beyond the largest bf16 propagate as in
    the fp32 matrix instruction; zeros, tiny values and an image whose other
    workgroups see ordinary values keep theirs."""
    from paper_2112_10603_amd import op_conv
    print(f"case direct fp32 extremes s={stride} T={transposed} cout={cout}", flush=True)
    x, wt, b = _data(64, cout, 1, 40, 40, transposed, 3)
    x[0, 3, 5, 5] = np.inf
    x[0, 9, 6, 30] = -np.inf
    x[0, 1, 30, 7] = np.nan
    x[0, 2, 33, 33] = 3.4028e38  # rounds to infinity in bf16
    x[0, :, 20:24, 20:24] = 1e-36
    x[0, :, 10:14, 20:24] = 0
    xd = torch.from_numpy(x).cuda()
    kw = dict(stride=max(stride, 1), transposed=transposed, precision="fp32")
    got = op_conv(xd, wt, b, **kw).cpu().numpy()
    ref = op_conv(xd, wt, b, n_tile=32, **kw).cpu().numpy()
    np.testing.assert_array_equal(np.isnan(got), np.isnan(ref))
    np.testing.assert_array_equal(np.isposinf(got), np.isposinf(ref))
    np.testing.assert_array_equal(np.isneginf(got), np.isneginf(ref))
    assert np.isnan(ref).any() and np.isinf(ref).any()
    fin = np.isfinite(ref)
    err = np.abs(got[fin].astype(np.float64) - ref[fin])
    # two fp32 evaluations, each within 2e-5 of the sum of |terms| (values of
    # order 1, or of the one huge activation times a weight)
    assert np.all(err <= 4e-5 * np.maximum(np.abs(ref[fin].astype(np.float64)), 8.0))
