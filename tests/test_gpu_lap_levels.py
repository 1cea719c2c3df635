"""Eq. 3 loss at the sizes where its launches change: edges of the reduce
tiles (64 x 8 outputs), the level at which the one-workgroup passes take over
(at most 16384 samples per plane), images whose coarsest level is too large
for them, single-quad remainders, and calls from several threads at once."""
import threading

import numpy as np
import pytest
import torch

from oracle import laploss as LL
from tests.test_gpu_lap import DEV, _gpu, _sign_safe_mask

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,h,w", [
    (1, 33, 33), (2, 34, 33),        # smallest: everything after level 1 in one workgroup
    (1, 127, 129), (1, 130, 257),    # 64 / 65 columns and 64 / 65 rows of level 1
    (1, 255, 256), (1, 257, 255),    # level 1 of 16384 samples, and just above
    (2, 145, 511),                   # level 1 handled by launches, level 2 by one workgroup
    (1, 2049, 2050),                 # level 4 above 16384 samples: no one-workgroup pass
])
def test_lap_loss_level_edges(n, h, w):
    print(f"case lap levels n={n} {h}x{w}", flush=True)
    rng = np.random.default_rng(h * 7 + w)
    x = rng.random((n, 3, h, w)).astype(np.float32)
    gt = rng.random((n, 3, h, w)).astype(np.float32)
    loss, g = _gpu(x, gt)
    for i in range(n):
        xi, gi = x[i].astype(np.float64), gt[i].astype(np.float64)
        ref = LL.lap_loss(xi, gi)
        # bounds as for the other sizes: fp32 rounding of |L| (2e-6 of the
        # loss) and of the gradient's two separable passes (1e-5 of its scale)
        assert abs(loss[i] - ref) <= 2e-6 * ref, (i, loss[i], ref)
        gref = LL.lap_loss_grad(xi, gi)
        m = _sign_safe_mask(xi - gi)
        assert np.abs(g[i].astype(np.float64) - gref)[m].max() <= 1e-5 * np.abs(gref).max()


def test_lap_loss_threads_and_streams():
    """Calls that overlap in time on several threads and streams give the
    results of the same calls one after another."""
    from paper_2112_10603_amd import lap_loss
    print("case lap threads", flush=True)
    shapes = [(1, 64, 80), (3, 100, 75), (2, 256, 300), (1, 40, 500)]
    data = [(torch.rand((n, 3, h, w), device=DEV), torch.rand((n, 3, h, w), device=DEV)) for n, h, w in shapes]
    want = [lap_loss(x, gt, grad=True) for x, gt in data]
    torch.cuda.synchronize()
    bad = []

    def work(k):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for r in range(6):
                i = (k + r) % len(data)
                loss, g = lap_loss(*data[i], grad=True)
                s.synchronize()
                if not (torch.equal(loss, want[i][0]) and torch.equal(g, want[i][1])):
                    bad.append((k, r, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad
