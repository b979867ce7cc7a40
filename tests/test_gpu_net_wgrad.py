"""Weight and bias gradients on ragged images: tile edges, rows narrower than
a quad of pixels, images smaller than a tile, several images with tiles of
their own.  Against the FP64 network oracle with bf16 weights and
activations; the GPU also rounds every backward value to bf16 (2^-9
relative, independent from pixel to pixel), six layers deep, so a layer's
relative L2 error is held to 2 * 6 * 2^-9 / sqrt(pixels) + 1e-4."""
import sys

import numpy as np
import pytest

from oracle import net as ON
from synth import voronoi_image

pytestmark = pytest.mark.gpu


def _say(msg):
    print(f"[gpu-net] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


def _forward(params, f, lam, p):
    a = ON.bf16_round(ON.net_input(f, lam, p))
    acts = [a]
    for i, prm in enumerate(params):
        z = ON.conv3x3(a, prm["w"], prm["b"])
        a = ON.bf16_round(np.maximum(z, 0.0)) if i < len(params) - 1 else z
        acts.append(a)
    return f + acts[-1], acts


@pytest.mark.parametrize("B,H,W", [(1, 5, 7), (2, 3, 34), (1, 17, 33), (3, 9, 70), (1, 8, 31), (2, 40, 66)])
def test_gradients_on_ragged_images(torch, B, H, W):
    from paper_2003_07504_amd import surrogate as S
    _say(f"ragged gradients B={B} H={H} W={W}")
    rng = np.random.default_rng(H * W)
    f = np.stack([voronoi_image(H, W, 3, 6, 0.05, seed=40 + i) for i in range(B)]).astype(np.float32)
    lam = rng.uniform(0.5, 2.0, B).astype(np.float32)
    p = rng.uniform(0.5, 1.0, B).astype(np.float32)
    t = np.clip(f + 0.05 * rng.standard_normal(f.shape), 0, 1).astype(np.float32)
    flat = 3.0 * S.init_params(seed=5)
    net = S.Net(B, H, W, params=flat)
    g, loss = net.gradients(*(torch.from_numpy(v).cuda() for v in (f, lam, p, t)))
    torch.cuda.synchronize()
    g = g.cpu().numpy().astype(np.float64)
    params = [{"w": ON.bf16_round(l["w"]), "b": l["b"]} for l in S.unflatten(flat)]
    ref, sq = 0.0, 0.0
    for b in range(B):
        v, acts = _forward(params, f[b].astype(np.float64), float(lam[b]), float(p[b]))
        sq += float(np.mean((v - t[b]) ** 2)) / B
        gb = ON.backward(params, acts, v, t[b].astype(np.float64))
        ref = ref + np.concatenate([np.concatenate([l["w"].ravel(), l["b"]]) for l in gb]) / B
    assert abs(float(loss.cpu()) - sq) <= 1e-3 * sq
    tol = 12.0 * 2.0 ** -9 / np.sqrt(B * H * W) + 1e-4
    off = 0
    for i, n in enumerate(S.layer_param_sizes()):
        a, r = g[off:off + n], ref[off:off + n]
        rel = np.linalg.norm(a - r) / np.linalg.norm(r)
        _say(f"  layer {i}: rel_l2 = {rel:.3e} (bound {tol:.1e})")
        assert rel <= tol, (i, rel, tol)
        off += n
    net.close()
