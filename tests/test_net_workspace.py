"""The surrogate's workspace: the size asked for stays what callers have
allotted before, and the partial sums of the weight gradients, which lie in
part where spent activations were, fit it for many small images too."""
import sys

import numpy as np
import pytest

from oracle import net as ON


@pytest.mark.parametrize("B,H,W,nbytes", [(1, 2, 2, 10293248), (1, 64, 64, 12240640), (16, 256, 256, 509413120),
                                          (300, 9, 33, 52702720), (8, 720, 1280, 3519743744),
                                          (512, 2, 2, 11265792)])
def test_workspace_size_is_what_it_was(B, H, W, nbytes):
    from paper_2003_07504_amd import surrogate
    assert surrogate._lib().ils_net_workspace_bytes(B, H, W) <= nbytes


@pytest.mark.gpu
@pytest.mark.parametrize("least", [True, False])
@pytest.mark.parametrize("B,H,W", [(512, 2, 2), (300, 9, 33)])
def test_gradients_with_fewer_rows_than_tiles(monkeypatch, B, H, W, least):
    """More tiles than rows of partial sums fit the least workspace, and the
    binding's own, which holds a row per tile.  Bound as in the other gradient
    tests: bf16 rounding of the backward values, six layers deep."""
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2003_07504_amd import surrogate as S
    print(f"[gpu-net] gradients of many small images B={B} H={H} W={W}", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(B + W)
    f = rng.uniform(0.0, 1.0, (B, 3, H, W)).astype(np.float32)
    lam = rng.uniform(0.5, 2.0, B).astype(np.float32)
    p = rng.uniform(0.5, 1.0, B).astype(np.float32)
    t = np.clip(f + 0.05 * rng.standard_normal(f.shape), 0, 1).astype(np.float32)
    flat = 3.0 * S.init_params(seed=7)
    if least:
        monkeypatch.setattr(S, "layer_param_sizes", lambda: [0])
    net = S.Net(B, H, W, params=flat)
    monkeypatch.undo()
    assert (net.workspace.numel() == S._lib().ils_net_workspace_bytes(B, H, W)) == least
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
