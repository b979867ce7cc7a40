"""Sizes whose transform lengths are not among the tuned ones, against the
FP64 oracle (the parity bar of the other sizes: max-abs 1e-4, relative L2
1e-5): odd row lengths, the smallest and the longest splits, one-row-band
and ragged-band frames, and the four lengths left to the runtime-length
passes, alone and together with a compiled one.  And the column tile that a
rule picks by the amount of work does not change a bit: a frame alone
(narrow tile) equals the same frame in a batch of many (wide tile)."""
import sys

import numpy as np
import pytest

from oracle import ils as O
from synth import voronoi_image

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.fixture(scope="module")
def ils(torch):
    from paper_2003_07504_amd import ils as m
    return m


@pytest.mark.parametrize("H,W,C,welsch", [
    (3, 6, 2, False), (5, 10, 1, True), (9, 18, 1, False), (27, 150, 1, False), (125, 54, 3, True),
    (81, 250, 1, False), (300, 486, 1, True), (405, 1350, 1, False), (600, 800, 3, True), (1200, 1600, 1, False),
    (1875, 24, 1, False), (24, 3750, 1, True), (4050, 20, 1, False), (20, 8100, 1, False), (3456, 12, 1, False),
    (12, 7776, 1, False), (2187, 20, 1, False), (30, 8000, 1, True), (3125, 12, 1, False), (4000, 6, 1, False)])
def test_size_parity(torch, ils, H, W, C, welsch):
    _say(f"size H={H} W={W} C={C} welsch={welsch}")
    f = voronoi_image(H, W, C, max(4, H * W // 5000), 0.05, seed=H + W)
    plan = ils.Plan(H, W, C)
    ft = torch.from_numpy(f).cuda()
    if welsch:
        u = plan.smooth_welsch(ft, 20.0, 10 / 255, 4)
        ref = np.stack([O.ils_welsch(f[c].astype(np.float64), 20.0, 10 / 255, 4) for c in range(C)])
    else:
        u = plan.smooth(ft, 1.0, 0.8, 1e-4, 4)
        ref = O.ils_channels(f.astype(np.float64), 1.0, 0.8, 1e-4, 4)
    torch.cuda.synchronize()
    assert plan.last_error() == 0
    d = u.cpu().numpy().astype(np.float64) - ref
    mx, rel = float(np.max(np.abs(d))), float(np.linalg.norm(d) / np.linalg.norm(ref))
    _say(f"  max {mx:.2e} rel {rel:.2e}")
    assert mx <= 1e-4 and rel <= 1e-5, (mx, rel)
    plan.close()


@pytest.mark.parametrize("H,W,n", [(256, 256, 40), (450, 600, 12), (60, 54, 64), (96, 1000, 24)])
def test_column_tile_rule_keeps_the_bits(torch, ils, H, W, n):
    _say(f"tile rule H={H} W={W} n={n}")
    fs = [torch.from_numpy(voronoi_image(H, W, 1, 8, 0.05, seed=300 + i)).cuda() for i in range(n)]
    plan = ils.Plan(H, W, 1, max_frames=n)
    outs = plan.smooth_batch([(f, 1.0 + 0.01 * i, 0.8, 1e-4, 3) for i, f in enumerate(fs)])
    for i in (0, n // 2, n - 1):
        one = plan.smooth(fs[i], 1.0 + 0.01 * i, 0.8, 1e-4, 3)
        torch.cuda.synchronize()
        assert torch.equal(one, outs[i]), i
    assert plan.last_error() == 0
    plan.close()
