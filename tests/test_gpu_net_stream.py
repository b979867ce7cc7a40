"""Inference streams strips of the image through all six layers in one launch;
a call in place runs layer by layer.  Both sum every product in the same
order, so they give the same bits, whatever the number of strips, of
segments down an image and of images: strips of exactly one, one more than
one and several widths, images smaller than the network's reach, odd row
counts (a last pair with one row), more units than compute units."""
import sys

import pytest

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-net] {msg}", flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("B,H,W", [(1, 2, 2), (1, 3, 54), (2, 7, 55), (1, 33, 109), (3, 61, 162), (1, 500, 56),
                                   (1, 1, 0), (40, 24, 400), (1, 1080, 130)])
def test_streamed_forward_equals_layers(B, H, W):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_07504_amd import surrogate as S
    if W == 0:
        with pytest.raises(ValueError):
            S.Net(B, H, W)
        return
    _say(f"stream B={B} H={H} W={W}")
    g = torch.Generator(device="cuda").manual_seed(B + H + W)
    f = torch.rand((B, 3, H, W), generator=g, device="cuda")
    lam = torch.rand(B, generator=g, device="cuda") + 0.5
    p = 0.5 * torch.rand(B, generator=g, device="cuda") + 0.5
    net = S.Net(B, H, W, params=3.0 * S.init_params(seed=4))
    v = net.forward(f, lam, p)
    inplace = f.clone()
    net.forward(inplace, lam, p, out=inplace)
    torch.cuda.synchronize()
    assert torch.isfinite(v).all()
    assert torch.equal(v, inplace)
    net.close()
