"""Served batches of several camera sizes whose convolutions are too large for
the direct-weight kernel, so that layers run as one launch over two or more
size groups: every view equals the view computed alone, bit for bit."""
import time

import numpy as np
import pytest
import torch

from synth import scenes
from synth.weights import write_weights_file

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


# Views of a size in one batch: 4 of 352 x 512 are 45056 pixels of the last
# stage's 256-channel layers (352 tiles of 128 x 256, more than the 256 that
# the direct kernel takes), 4 of 368 x 480 are 44160; one of 720 x 1280 is
# 57600.
@pytest.mark.parametrize("precision", ["bf16", "fp8"])
@pytest.mark.parametrize("sizes", [[(352, 512)] * 4 + [(361, 475)] * 4, [(720, 1280), (704, 1264), (352, 512), (48, 64)]])
def test_grouped_launches(tmp_path, precision, sizes):
    from paper_2112_10603_amd import Net
    print(f"case serving groups {precision} {sizes}", flush=True)
    path = write_weights_file(str(tmp_path / "w.ffvw"), seed=0)
    served = Net(path, precision, 0, hbm_budget_bytes=32 << 30, tick_ms=5.0, max_batch_views=len(sizes))
    alone = Net(path, precision, 0)
    if precision == "fp8":
        cal = scenes.random_pair(99, 96, 96)
        for net in (served, alone):
            net.calibrate(cal[0].to(DEV), cal[1].to(DEV), 0.5)
    cams, ids = {}, {}
    for size in dict.fromkeys(sizes):
        arc = scenes.camera_arc(len(ids), *size, 2, 128, (3.0, 9.0), 4.0, 0.01).to(DEV)
        cams[size] = (arc[0].contiguous(), arc[1].contiguous())
        ids[size] = 2 * len(ids)
        for i in range(2):
            served.register_camera(ids[size] + i, cams[size][i])
    rng = np.random.default_rng(4)
    ts = [float(rng.uniform(0, 1)) for _ in sizes]
    outs = [torch.full((3,) + s, -1.0, device=DEV) for s in sizes]
    tickets = served.submit_many([(ids[s], ids[s] + 1, t, o) for s, t, o in zip(sizes, ts, outs)])
    done = {}
    t0 = time.time()
    while len(done) < len(tickets) and time.time() - t0 < 60:
        for tk in tickets:
            if tk not in done:
                r = served.poll(tk)
                if r is not None:
                    done[tk] = r
        time.sleep(0.001)
    assert len({done[tk]["t_launch"] for tk in tickets}) == 1
    torch.cuda.synchronize()
    for k, (s, t, o) in enumerate(zip(sizes, ts, outs)):
        assert torch.equal(o, alone.interpolate([cams[s]], [t])[0, 0]), (k, s)
    alone.close()
    served.close()
