"""Many short or narrow images run layer by layer where strips would be mostly
waste: the same bits as the strips that a part of the batch takes on its own,
and not slower than the layers that a call in place takes."""
import sys

import pytest

pytestmark = pytest.mark.gpu

# (images, rows, columns, images of a part that runs as strips)
SIZES = [(512, 8, 55, 32), (267, 327, 5, 40), (479, 3, 1533, 4), (512, 2, 2, 64), (300, 33, 64, 20)]


def _net(B, H, W):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_07504_amd import surrogate as S
    print(f"[gpu-net] narrow B={B} H={H} W={W}", flush=True)
    sys.stdout.flush()
    g = torch.Generator(device="cuda").manual_seed(B + H + W)
    f = torch.rand((B, 3, H, W), generator=g, device="cuda")
    lam = torch.rand(B, generator=g, device="cuda") + 0.5
    p = 0.5 * torch.rand(B, generator=g, device="cuda") + 0.5
    return torch, S.Net(B, H, W, params=3.0 * S.init_params(seed=4)), f, lam, p


@pytest.mark.parametrize("B,H,W,part", SIZES)
def test_layers_and_strips_give_the_same_bits(B, H, W, part):
    torch, net, f, lam, p = _net(B, H, W)
    v = net.forward(f, lam, p)
    for b in range(0, B, part):
        e = min(b + part, B)
        w = net.forward(f[b:e].contiguous(), lam[b:e].contiguous(), p[b:e].contiguous())
        assert torch.equal(v[b:e], w), b
        if b >= 3 * part:
            break
    net.close()


@pytest.mark.parametrize("B,H,W", [(267, 327, 5), (479, 3, 1533)])
def test_not_slower_than_in_place(B, H, W):
    torch, net, f, lam, p = _net(B, H, W)
    out = torch.empty_like(f)

    def best(o):
        t = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(8):
                net.forward(f, lam, p, out=o)
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    best(out)
    assert best(out) <= 1.2 * best(f)
    net.close()
