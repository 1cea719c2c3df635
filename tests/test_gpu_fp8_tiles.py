"""FP8 launches on the direct-weight kernel and on the other tiles: a view
equals itself in batches whose layers cross the limits of the tile rule, bit
for bit."""
import pytest
import torch

from synth import scenes
from synth.weights import write_weights_file

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


@pytest.fixture(scope="module")
def net(tmp_path_factory):
    from paper_2112_10603_amd import Net
    net = Net(write_weights_file(str(tmp_path_factory.mktemp("w8") / "w0.ffvw"), seed=0), "fp8", 0)
    cal = scenes.random_pair(99, 96, 96)
    net.calibrate(cal[0].to(DEV), cal[1].to(DEV), 0.5)
    yield net
    net.close()


# Workgroups of the 64 x 64 direct tile (limit 512) of one view and of the
# batch. 180 x 320: stage 2's 256-channel layers (48 x 80) 240 and, in 4
# views, 960, its transposed conv 480 and 1920; stage 1's (24 x 40) 60 and, in
# 12 views, 720. 360 x 640: stage 2's (92 x 160) are past the limit alone; 120
# halo tiles of 256 pixels x 128 columns alone (limit 256) and, in 6 views, 720.
@pytest.mark.parametrize("h,w,n", [(180, 320, 4), (180, 320, 12), (360, 640, 2), (360, 640, 6), (77, 301, 16)])
def test_fp8_view_equals_itself_in_a_batch(net, h, w, n):
    print(f"case fp8 tiles {h}x{w} x {n}", flush=True)
    arc = scenes.camera_arc(h + n, h, w, 2, 128, (3.0, 10.0), 6.0, 0.01).to(DEV)
    pair = (arc[0].contiguous(), arc[1].contiguous())
    ts = [(k + 1) / (n + 1) for k in range(n)]
    batch = net.interpolate([pair], ts)[0]
    for k in (0, n // 2, n - 1):
        assert torch.equal(net.interpolate([pair], [ts[k]])[0, 0], batch[k]), k


def test_fp8_direct_equals_table_tiles(net, tmp_path):
    """The FP8 layers of an 180 x 320 view on explicit tiles, through a tuning
    table, against the direct kernel."""
    print("case fp8 direct against explicit tiles", flush=True)
    arc = scenes.camera_arc(8, 180, 320, 2, 128, (3.0, 10.0), 6.0, 0.01).to(DEV)
    pairs = [(arc[0].contiguous(), arc[1].contiguous())]
    ref = net.interpolate(pairs, [0.5])
    rows = []
    for s in range(3):  # padded 192 x 320, quarter to full size, divided by 4
        h, w = 12 << s, 20 << s
        rows += [f"vib{s}.conv{i} 1 {h} {w} 1 256 16 1" for i in range(2, 9)]
        rows.append(f"vib{s}.convT1 1 {h} {w} 1 128 16 1")
    path = tmp_path / "t.txt"
    path.write_text("\n".join(rows) + "\n")
    assert net.load_tuning(str(path)) == len(rows)
    assert torch.equal(net.interpolate(pairs, [0.5]), ref)
    # back to the rule's tiles for the tests that share the net
    path.write_text("\n".join(r.rsplit(" ", 3)[0] + " direct 16 1" for r in rows) + "\n")
    assert net.load_tuning(str(path)) == len(rows)
    assert torch.equal(net.interpolate(pairs, [0.5]), ref)
