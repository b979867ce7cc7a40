"""Backward pass where a block walks several tiles, where every block has one,
and on the smallest image.  Against the FP64 network oracle with bf16 weights
and activations; the GPU also rounds every backward value to bf16 (2^-9
relative, independent from pixel to pixel), six layers deep, so a layer's
relative L2 error is held to 2 * 6 * 2^-9 / sqrt(pixels) + 1e-4."""
import sys

import numpy as np
import pytest

from oracle import net as ON

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("B,H,W", [(3, 200, 200), (1, 64, 64), (1, 2, 2)])
def test_backward_over_the_tiles(torch, B, H, W):
    from paper_2003_07504_amd import surrogate as S
    print(f"[gpu-net] backward B={B} H={H} W={W}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(B * H)
    f = rng.uniform(0.0, 1.0, (B, 3, H, W)).astype(np.float32)
    lam = rng.uniform(0.5, 2.0, B).astype(np.float32)
    p = rng.uniform(0.5, 1.0, B).astype(np.float32)
    t = np.clip(f + 0.05 * rng.standard_normal(f.shape), 0, 1).astype(np.float32)
    flat = 3.0 * S.init_params(seed=6)
    net = S.Net(B, H, W, params=flat)
    g, loss = net.gradients(*(torch.from_numpy(v).cuda() for v in (f, lam, p, t)))
    torch.cuda.synchronize()
    g = g.cpu().numpy().astype(np.float64)
    params = [{"w": ON.bf16_round(l["w"]), "b": l["b"]} for l in S.unflatten(flat)]
    ref, sq = 0.0, 0.0
    for b in range(B):
        x = f[b].astype(np.float64)
        a = ON.bf16_round(ON.net_input(x, float(lam[b]), float(p[b])))
        acts = [a]
        for i, prm in enumerate(params):
            z = ON.conv3x3(a, prm["w"], prm["b"])
            a = ON.bf16_round(np.maximum(z, 0.0)) if i < len(params) - 1 else z
            acts.append(a)
        v = x + acts[-1]
        sq += float(np.mean((v - t[b]) ** 2)) / B
        gb = ON.backward(params, acts, v, t[b].astype(np.float64))
        ref = ref + np.concatenate([np.concatenate([l["w"].ravel(), l["b"]]) for l in gb]) / B
    assert abs(float(loss.cpu()) - sq) <= 1e-3 * sq
    tol = 12.0 * 2.0 ** -9 / np.sqrt(B * H * W) + 1e-4
    off = 0
    for i, n in enumerate(S.layer_param_sizes()):
        rel = np.linalg.norm(g[off:off + n] - ref[off:off + n]) / np.linalg.norm(ref[off:off + n])
        print(f"[gpu-net]   layer {i}: rel_l2 = {rel:.3e} (bound {tol:.1e})", flush=True)
        assert rel <= tol, (i, rel, tol)
        off += n
    net.close()
