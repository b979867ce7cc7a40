"""Penalties and images far from unit size.  The smoother is equivariant: an
image times t with gamma t (Welsch), or with eps t^2 and lambda t^(2-p)
(Charbonnier), gives the result times t.  For t a power of two the Welsch
arithmetic is the same up to exponents, so the bits agree; the Charbonnier
penalty's constants round differently where the iterate's scale is at its
limit, so that is held to the parity bar against the FP64 oracle."""
import sys

import numpy as np
import pytest

from oracle import ils as O
from synth import voronoi_image

pytestmark = pytest.mark.gpu

MAX_ABS = 1e-4
REL_L2 = 1e-5
# compiled passes, and a column length on the runtime-length passes
SIZES = [(64, 96), (2187, 8)]


def _say(msg):
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("H,W", SIZES)
@pytest.mark.parametrize("k", [-70, -44, -20, 20, 44, 70])
def test_welsch_is_equivariant(torch, H, W, k):
    from paper_2003_07504_amd import ils
    _say(f"Welsch times 2^{k}, {H}x{W}")
    f = voronoi_image(H, W, 1, 20, 0.05, seed=3)
    t = np.float32(2.0 ** k)
    plan = ils.Plan(H, W, 1)
    a = plan.smooth_welsch(torch.from_numpy(f).cuda(), 20.0, float(np.float32(10 / 255)), 5)
    b = plan.smooth_welsch(torch.from_numpy(f * t).cuda(), 20.0, float(np.float32(10 / 255) * t), 5)
    torch.cuda.synchronize()
    assert torch.equal(a * float(t), b)
    plan.close()


@pytest.mark.parametrize("H,W", SIZES)
@pytest.mark.parametrize("k", [-56, -30, 30, 56])
def test_charbonnier_keeps_parity_at_every_width(torch, H, W, k):
    from paper_2003_07504_amd import ils
    _say(f"Charbonnier times 2^{k}, {H}x{W}")
    f = voronoi_image(H, W, 1, 20, 0.05, seed=4)
    t = np.float32(2.0 ** k)
    eps = float(np.float32(1e-4) * t * t)
    ref = O.ils_channels(f.astype(np.float64), 1.0, 1.0, 1e-4, 4)
    plan = ils.Plan(H, W, 1)
    u = plan.smooth(torch.from_numpy(f * t).cuda(), float(t), 1.0, eps, 4)
    torch.cuda.synchronize()
    d = u.cpu().numpy().astype(np.float64) / float(t) - ref
    assert np.max(np.abs(d)) <= MAX_ABS and np.linalg.norm(d) <= REL_L2 * np.linalg.norm(ref)
    plan.close()


@pytest.mark.parametrize("gamma", [1e-30, 1e30])
def test_welsch_limits(torch, gamma):
    """gamma far below any difference leaves mu = c g, so u = f; far above,
    mu = 0 and the solve is the quadratic filter of p = 2."""
    from paper_2003_07504_amd import ils
    f = voronoi_image(32, 48, 1, 8, 0.05, seed=5)
    plan = ils.Plan(32, 48, 1)
    x = torch.from_numpy(f).cuda()
    u = plan.smooth_welsch(x, 2.0, gamma, 3).cpu().numpy().astype(np.float64)
    # p = 2: c0 = 2, so lambda c0 / 2 = lambda as for Welsch
    ref = f.astype(np.float64) if gamma < 1 else O.ils_channels(f.astype(np.float64), 2.0, 2.0, 1e-4, 3)
    assert np.max(np.abs(u - ref)) <= MAX_ABS and np.linalg.norm(u - ref) <= REL_L2 * np.linalg.norm(ref)
    plan.close()


@pytest.mark.parametrize("H,W", SIZES)
@pytest.mark.parametrize("eps,size", [(1e-36, 1e22), (1e36, 1e-22)])
def test_charbonnier_limits(torch, H, W, eps, size):
    """Images far larger than sqrt(eps) keep mu = c g, so u = f; far smaller,
    mu = 0.  The iterate's own scale must not leave float32's range."""
    from paper_2003_07504_amd import ils
    _say(f"Charbonnier eps={eps:g} image size {size:g}, {H}x{W}")
    f = (voronoi_image(H, W, 1, 20, 0.05, seed=6) * np.float32(size)).astype(np.float32)
    lam = 2.0 * np.sqrt(eps)  # kappa = lambda c0 / 2 = 1 for p = 1
    ref = O.ils_channels(f.astype(np.float64), float(np.float32(lam)), 1.0, float(np.float32(eps)), 3)
    plan = ils.Plan(H, W, 1)
    u = plan.smooth(torch.from_numpy(f).cuda(), lam, 1.0, eps, 3)
    torch.cuda.synchronize()
    d = u.cpu().numpy().astype(np.float64) - ref
    assert np.max(np.abs(d)) <= MAX_ABS * size and np.linalg.norm(d) <= REL_L2 * np.linalg.norm(ref)
    plan.close()
