"""Results written to an image that starts at an odd float (a view into a
larger buffer): the same bits as into an aligned one, and nothing beside it."""
import sys

import pytest

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


def _odd(torch, shape):
    """(buffer, view of `shape` that starts at its second float)."""
    n = 1
    for s in shape:
        n *= s
    buf = torch.full((n + 2,), -7.0, device="cuda")
    return buf, buf[1:n + 1].view(*shape)


# several band shapes, a three-stage column length, a ragged last band, and the runtime-length passes
@pytest.mark.parametrize("H,W,C", [(64, 96, 1), (450, 600, 3), (81, 54, 2), (1080, 1920, 1), (2187, 8, 1)])
@pytest.mark.parametrize("what", ["smooth", "detail", "welsch", "batch"])
def test_odd_output(torch, H, W, C, what):
    from paper_2003_07504_amd import ils
    _say(f"odd output {what} {H}x{W}x{C}")
    f = torch.from_numpy(voronoi_image(H, W, C, 30, 0.05, seed=8)).cuda()
    plan = ils.Plan(H, W, C, max_frames=2)
    run = {"smooth": lambda o: plan.smooth(f, 1.0, 0.8, 1e-4, 2, out=o),
           "detail": lambda o: plan.detail_enhance(f, 1.0, 0.8, 1e-4, 2, 3.0, out=o),
           "welsch": lambda o: plan.smooth_welsch(f, 20.0, 0.04, 2, out=o),
           "batch": lambda o: plan.smooth_batch([(f, 1.0, 0.8, 1e-4, 2), (f, 0.5, 0.9, 1e-4, 2)],
                                                outs=[o, torch.empty_like(f)])}[what]
    want = torch.empty_like(f)
    run(want)
    buf, view = _odd(torch, f.shape)
    assert view.data_ptr() % 8 == 4
    run(view)
    torch.cuda.synchronize()
    assert plan.last_error() == 0
    assert torch.equal(view, want)
    assert buf[0].item() == -7.0 and buf[-1].item() == -7.0
    plan.close()


@pytest.mark.parametrize("H,W", [(96, 64), (81, 54)])
@pytest.mark.parametrize("K", [1, 3])
def test_odd_tone_map(torch, H, W, K):
    from paper_2003_07504_amd import ils
    _say(f"odd tone map {H}x{W} K={K}")
    f = 10.0 ** (3.0 * torch.from_numpy(voronoi_image(H, W, 3, 20, 0.05, seed=9)).cuda())
    plan = ils.Plan(H, W, 3)
    lams = [0.125, 1.0, 8.0][:K]
    want = plan.tone_map_multiscale(f, lams, 1.0, 1e-4, 3, 100.0, [1.0] * K)
    buf, view = _odd(torch, f.shape)
    plan.tone_map_multiscale(f, lams, 1.0, 1e-4, 3, 100.0, [1.0] * K, out=view)
    torch.cuda.synchronize()
    assert torch.equal(view, want)
    assert buf[0].item() == -7.0 and buf[-1].item() == -7.0
    plan.close()
