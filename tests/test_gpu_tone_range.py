"""Tone mapping of radiances whose gain is near the end of float32: the
logarithm is taken relative to a power of two, which must not push the gain's
exponential out of range.  Bound: the base's max-abs bar (1e-4 of the
logarithm's range) times detail + 1, as a relative error of the result."""
import sys

import numpy as np
import pytest

from oracle import ils as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bright,spot,detail", [(1e16, 1e4, 4.0), (1e16, 1e5, 3.5), (1e20, 2.2e4, 3.5)])
def test_gain_near_the_end_of_the_range(bright, spot, detail):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_07504_amd import ils
    print(f"[gpu] tone map of {bright:g} with spots of {spot:g}, detail {detail}", flush=True)
    sys.stdout.flush()
    y = np.full((64, 64), bright, dtype=np.float32)
    y[:, :16] = 1e-6
    y[20, 8] = y[40, 9] = spot
    f = np.stack([y, y, y])
    ref = O.tone_map(f.astype(np.float64), 4.0, 2.0, 1e-4, 1, contrast=float(np.float32(1.0001)), detail=detail)
    plan = ils.Plan(64, 64, 3)
    out = plan.tone_map(torch.from_numpy(f).cuda(), 4.0, 2.0, 1e-4, 1, 1.0001, detail)
    torch.cuda.synchronize()
    got = out.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    span = np.log(bright / 1e-6)
    assert np.max(np.abs(got / ref - 1.0)) <= 1e-4 * span * (detail + 1.0)
    plan.close()
