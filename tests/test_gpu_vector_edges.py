"""Branches that a size or an address selects: column tiles of the three-stage
pass of every width, the rule's tile widths, and the element-by-element forms of
the kernels that take four values at a time where they can."""
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


# heights whose 12-column tile fits 1024 lanes; padded rows of 336 columns (28
# tiles of 12), and of 272 and 496 (a ragged last one)
@pytest.mark.parametrize("H,W,C", [(480, 640, 3), (512, 512, 1), (640, 960, 1)])
def test_three_stage_tiles_are_bitwise_equal(torch, ils, H, W, C):
    nr, nc = ils.shape_variants(H, W)
    _say(f"three-stage tiles {H}x{W}x{C}: {nr} row x {nc} column shapes")
    assert nc == 4
    f = torch.from_numpy(voronoi_image(H, W, C, 60, 0.05, seed=12)).cuda()
    plan = ils.Plan(H, W, C)
    ref = None
    for c in range(nc):
        plan.set_shapes(H, W, C, 0, c)
        u = plan.smooth(f, 1.0, 0.8, 1e-4, 3)
        torch.cuda.synchronize()
        assert plan.last_error() == 0
        if ref is None:
            ref = u
        assert torch.equal(u, ref), c
    plan.close()


def _rule_width(torch, W, channels, widths=(16, 12, 8, 4)):
    """The widest tile that makes 0.7 blocks per compute unit, else the narrowest."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ld = (W // 2 + 1 + 15) // 16 * 16
    for w in widths:
        if 10 * channels * -(-ld // w) >= 7 * cus:
            return w
    return widths[-1]


@pytest.mark.parametrize("n", [96, 192])
def test_rule_takes_wider_tiles_for_batches_bit_for_bit(torch, ils, n):
    H, W = 60, 54
    widths = (_rule_width(torch, W, 1), _rule_width(torch, W, n // 2))  # a frame, and a part of the batch
    _say(f"tiles of {widths} columns for one and {n // 2} frames of {H}x{W}")
    assert widths[0] < widths[1]
    fs = [torch.from_numpy(voronoi_image(H, W, 1, 8, 0.05, seed=300 + i)).cuda() for i in range(n)]
    plan = ils.Plan(H, W, 1, max_frames=n)
    outs = plan.smooth_batch([(f, 1.0 + 0.01 * i, 0.8, 1e-4, 3) for i, f in enumerate(fs)])
    for i in (0, n // 2 - 1, n // 2, n - 1):
        one = plan.smooth(fs[i], 1.0 + 0.01 * i, 0.8, 1e-4, 3)
        torch.cuda.synchronize()
        assert torch.equal(one, outs[i]), i
    plan.close()


@pytest.mark.parametrize("count", [1, 3, 4, 1023, 70001])
@pytest.mark.parametrize("oa,ob", [(0, 0), (1, 0), (0, 1), (1, 1), (2, 2)])
def test_rms_of_any_alignment(torch, ils, count, oa, ob):
    rng = np.random.default_rng(count)
    a, b = rng.uniform(0, 1, count + 4).astype(np.float32), rng.uniform(0, 1, count + 4).astype(np.float32)
    plan = ils.Plan(8, 8, 1)
    ta, tb = torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()
    r = plan.rms_diff([ta[oa:oa + count]], [tb[ob:ob + count]]).cpu().numpy()
    d = a[oa:oa + count].astype(np.float64) - b[ob:ob + count].astype(np.float64)
    want = np.sqrt(np.mean(d * d))
    assert abs(float(r[0]) - want) <= 2.0 ** -23 * want  # summed in double, rounded once
    plan.close()


@pytest.mark.parametrize("k", [0.0, 2.0])
def test_luminance_of_an_odd_plane(torch, ils, k):
    H, W = 81, 54  # 4374 values: no multiple of four
    f = voronoi_image(H, W, 3, 10, 0.05, seed=13)
    ref = O.ils_luminance(f.astype(np.float64), 1.0, 0.8, 1e-4, 4, k=k)
    plan = ils.Plan(H, W, 3)
    out = plan.smooth_luminance(torch.from_numpy(f).cuda(), 1.0, 0.8, 1e-4, 4, k).cpu().numpy().astype(np.float64)
    d = out - ref
    scale = max(1.0, abs(1.0 - k))
    assert np.max(np.abs(d)) <= 1e-4 * scale and np.linalg.norm(d) <= 1e-5 * scale * np.linalg.norm(ref)
    plan.close()
