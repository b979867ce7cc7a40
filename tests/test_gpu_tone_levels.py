"""Multi-scale tone mapping runs its levels as the channels of one sequence
of passes where the workspace and the output have room, in two groups where
the workspace holds two levels' spectra, and one after another in place or
when a level is the log-luminance itself.  Every route against the FP64
oracle (per-pixel relative error, the bound of the other tone-mapping tests:
5e-5), on planes that do and do not divide by four, a size of the
runtime-length passes, and radiance far from 1."""
import sys

import numpy as np
import pytest

from oracle import ils as O
from synth import hdr_image

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


LAMS = (0.125, 0.5, 2.0, 8.0)
WEIGHTS = (1.3, 1.2, 1.1, 1.0)


@pytest.mark.parametrize("H,W,K,room,in_place,zero,gain", [
    (64, 96, 3, "all", False, False, 1.0), (64, 96, 3, "min", False, False, 1.0), (64, 96, 4, "min", False, False, 1.0),
    (64, 96, 2, "min", False, False, 1e6), (64, 96, 3, "all", True, False, 1.0), (64, 96, 3, "all", False, True, 1.0),
    (81, 54, 4, "all", False, False, 1e-3), (81, 54, 3, "min", False, False, 1.0), (2187, 8, 3, "all", False, False, 1.0),
    (720, 1280, 3, "all", False, False, 1.0), (96, 90, 1, "all", False, False, 1.0)])
def test_level_routes(torch, H, W, K, room, in_place, zero, gain):
    from paper_2003_07504_amd import _lib, ils
    lams = list(LAMS[:K])
    if zero:
        lams[0] = 0.0
    _say(f"levels H={H} W={W} K={K} room={room} in_place={in_place} zero={zero} gain={gain}")
    f = (gain * hdr_image(H, W, K=max(4, H * W // 5000), seed=70 + H)).astype(np.float32)
    ref = O.tone_map_multiscale(f.astype(np.float64), lams, 1.0, 1e-4, 3, contrast=100.0, weights=WEIGHTS[:K])
    if room == "all":
        plan = ils.Plan(H, W, 4)
    else:
        plan = ils.Plan(H, W, 1, ws_bytes=int(_lib.load().ils_tone_map_multiscale_workspace_bytes(H, W, K)))
    ft = torch.from_numpy(f).cuda()
    out = ft if in_place else torch.full_like(ft, float("nan"))
    plan.tone_map_multiscale(ft, lams, 1.0, 1e-4, 3, 100.0, WEIGHTS[:K], out=out)
    torch.cuda.synchronize()
    assert plan.last_error() == 0
    rel = np.abs(out.cpu().numpy().astype(np.float64) - ref) / ref
    _say(f"  max rel {rel.max():.2e}")
    assert rel.max() < 5e-5, rel.max()
    if not in_place:
        assert torch.equal(ft, torch.from_numpy(f).cuda())
    plan.close()
