"""Texture adjoint where pixel runs share base texels: textures from one texel to several texels a pixel, repeat and
clamp, with and without the fused loss and its sum (which changes the block shape up to four layers), on views that end
inside a tile.  Gradients against the oracle's analytic adjoint, the loss sum to its FP64 bar."""
import numpy as np
import pytest

import oracle as O
import scenes as S
from vs_testlib import GRAD_RTOL, gpu_render, grad_rel_err, oracle_vis, say, small_mixed_scene

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 4, 5])
@pytest.mark.parametrize("wrap", [0, 1])
@pytest.mark.parametrize("tex", [1, 3, 8, 33, 200, 900])
def test_gradient_of_runs(k, wrap, tex):
    import torch
    assert torch.cuda.is_available()
    sc = small_mixed_scene(k=k, tex=tex, config=140 + k, sizes=((96, 80), (37, 53), (17, 130)))
    P, layers, views, vis, ws, _, texs = gpu_render(sc, wrap=wrap)
    seen = [oracle_vis(sc, views, vis, v) for v in range(len(sc.cameras))]
    gs = [S.upstream_grad(140 + k, c, v) for v, c in enumerate(sc.cameras)]
    target = [np.abs(g) for g in gs]
    flat = lambda xs: torch.from_numpy(np.concatenate([x.reshape(-1, 4) for x in xs]).astype(np.float32)).cuda()  # noqa: E731
    say(f"[gpu] runs k={k} wrap={wrap} tex={tex}")
    plain = P.render_backward(layers, texs, views, vis, ws, grad_rgba=flat(gs), wrap=wrap)
    sse = torch.zeros(1, dtype=torch.float64, device="cuda")
    fused = P.render_backward(layers, texs, views, vis, ws, target=flat(target), sse=sse, wrap=wrap)
    torch.cuda.synchronize()
    want_p, want_f, loss = [0.0] * k, [0.0] * k, 0.0
    for v, cam in enumerate(sc.cameras):
        img = O.shade(sc.layers, sc.textures, cam, seen[v], wrap=wrap)
        d = np.zeros_like(img)
        d[..., :3] = img[..., :3] - target[v][..., :3].astype(np.float64)
        loss += float((d ** 2).sum())
        for want, g in ((want_p, gs[v].astype(np.float64)), (want_f, 2.0 * d)):
            back = O.backward(sc.layers, sc.textures, cam, seen[v], grad_out=g, wrap=wrap)
            for l in range(k):
                want[l] = want[l] + back[l]
    for got, want in ((plain, want_p), (fused, want_f)):
        assert grad_rel_err([g.cpu().numpy().astype(np.float64) for g in got], want) <= GRAD_RTOL
    assert abs(sse.item() - loss) <= 1e-6 * loss
