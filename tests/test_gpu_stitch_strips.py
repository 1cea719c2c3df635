"""Cluster frames at the sizes where the kernel changes: tiles 64 pixels wide
and one short of it, more columns than a workgroup's threads, and views whose
alignment the wide loads cannot take."""
import numpy as np
import pytest
import torch

from oracle import stitch as S

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,H,W,shift", [
    (1, 5, 63, 0), (1, 5, 64, 0), (1, 3, 300, 0), (4, 6, 126, 0), (4, 6, 128, 0), (4, 10, 700, 1),
    (16, 8, 252, 0), (16, 8, 256, 0), (16, 12, 1100, 0), (64, 16, 504, 0), (64, 16, 512, 0), (64, 8, 2200, 0),
    (64, 8, 640, 2), (1, 4, 100, 1),
])
def test_stitch_strip_edges(n, H, W, shift):
    """`shift` floats before each view: 0 keeps 16-byte alignment."""
    from paper_2112_10603_amd import stitch_cluster
    print(f"case stitch strips n={n} {H}x{W} shift={shift}", flush=True)
    rng = np.random.default_rng(n * 100 + W)

    def views(k):
        host = [rng.random((3, H, W)).astype(np.float32) for _ in range(k)]
        dev = []
        for v in host:
            buf = torch.empty(3 * H * W + shift, dtype=torch.float32, device=DEV)
            buf[shift:] = torch.from_numpy(v.ravel())
            dev.append(buf[shift:].view(3, H, W))
        return host, dev

    (hr,), (hr_d,) = views(1)
    left, left_d = views(n)
    right, right_d = views(n)
    got = stitch_cluster(hr_d, left_d, right_d).cpu().numpy()
    ref = S.stitch_cluster(hr, left, right)
    # g * g fp32 additions of values in [0, 1] and one exact scaling
    assert np.abs(got.astype(np.float64) - ref).max() <= 1e-6
    np.testing.assert_array_equal(got[:, :, W:2 * W], hr)
