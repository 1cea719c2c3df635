"""Cluster frames of 16 views a side whose real view or frame is not 16-byte
aligned (the side views always are: others are refused)."""
import numpy as np
import pytest
import torch

from oracle import stitch as S

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _at(host, shift):
    buf = torch.empty(host.size + 4, dtype=torch.float32, device=DEV)
    view = buf[shift:shift + host.size].view(*host.shape)
    view.copy_(torch.from_numpy(host))
    return view


@pytest.mark.parametrize("H,W", [(8, 256), (12, 1100)])
@pytest.mark.parametrize("real,out", [(0, 0), (1, 0), (2, 0), (0, 1), (0, 3), (1, 1)])
def test_unaligned_real_view_and_frame(H, W, real, out):
    from paper_2112_10603_amd import stitch_cluster
    print(f"case stitch alignment {H}x{W} real={real} out={out}", flush=True)
    rng = np.random.default_rng(W + 10 * real + out)
    host = rng.random((33, 3, H, W)).astype(np.float32)
    left, right = ([_at(v, 0) for v in host[k:k + 16]] for k in (1, 17))
    frame = _at(np.full((3, H, 3 * W), -1.0, np.float32), out)
    got = stitch_cluster(_at(host[0], real), left, right, frame).cpu().numpy()
    ref = S.stitch_cluster(host[0], host[1:17], host[17:])
    # 16 fp32 additions of values in [0, 1] and one exact scaling
    assert np.abs(got.astype(np.float64) - ref).max() <= 1e-6
    np.testing.assert_array_equal(got[:, :, W:2 * W], host[0])


def test_unaligned_side_view_refused():
    from paper_2112_10603_amd import FfvError, stitch_cluster
    print("case stitch alignment refused", flush=True)
    host = np.zeros((3, 8, 256), np.float32)
    views = [_at(host, 0) for _ in range(32)]
    views[20] = _at(host, 1)
    with pytest.raises(FfvError) as e:
        stitch_cluster(_at(host, 0), views[:16], views[16:])
    assert e.value.code == -1
