"""The two launches of the preprocess backward (chain of the splats with rows, one stream over the parameters) at the
edges of their blocks, for every SH degree: one view against the oracle; several views against the views one by one;
the fused Adam update, small and with its loads past the caches, against stored gradients and the stand-alone step."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

from .parity_helpers import assert_grad_ok, gpu_render, grad3d_check, oracle_full, to_device

pytestmark = pytest.mark.gpu
LRS = {"means": 1e-4, "sh": 2e-3, "opacity_logits": 5e-2, "beta": 1e-3, "quats": 1e-3, "log_scales": 5e-3}


def _scene(n, degree, seed=70):
    return synth.scene_clusters(n, seed + degree, degree=degree, n_clusters=4).arrays()


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 64, 65, 257, 700])
def test_gradients_against_the_oracle(n, degree):
    print(f"[chain] n={n} degree={degree}", flush=True)
    sc = _scene(n, degree)
    cam = synth.orbit_camera(np.random.default_rng(3), 75, 61)
    dL = np.random.default_rng(4).standard_normal((61, 75, 3)).astype(np.float32)
    gpu = gpu_render(sc, degree, cam, O.FALLOFF_PHI, O.TILES_ELLIPSE, dL=dL)
    ref = oracle_full(sc, degree, cam, O.FALLOFF_PHI, O.TILES_ELLIPSE, dL=dL.astype(np.float64))
    for k in gpu["grads"]:
        assert_grad_ok(f"d{k}", grad3d_check(gpu["grads"][k], ref["grads"][k], ref["allow"][k]))


def _backward(t, cams, dLs, call):
    """Renders the views in one batch and calls call(*workspaces)."""
    s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
    p = G.params_struct(0, G.TILES_ELLIPSE)
    cs = [G.camera_struct(c) for c in cams]
    f = G.Frame.create(s.n, cams[0].width, cams[0].height, views=len(cams))
    f.ensure_keys(G.ges_preprocess_views(s, cs, p, f.splat_ws, True))
    img = torch.empty((len(cams), cams[0].height, cams[0].width, 3), device="cuda")
    G.ges_render_forward_views(s, cs, p, f.splat_ws, f.key_ws, f.num_keys, f.pixel_ws, img)
    call(s, cs, p, f.splat_ws, f.key_ws, f.pixel_ws, dLs)
    torch.cuda.synchronize()


@pytest.mark.parametrize("n,degree", [(65, 0), (257, 1), (300, 2), (1000, 3), (380_000, 3)],
                         ids=["65_d0", "257_d1", "300_d2", "1000_d3", "380k_d3_past_the_caches"])
@pytest.mark.parametrize("views", [1, 3, 6])   # up to 4 views travel with the first kernel, more by a copy
def test_views_and_fused_update(n, degree, views):
    """Stored gradients of a batch are the views' gradients added in view order, also onto what the buffers held;
    the fused update takes the same bits as the stand-alone one."""
    print(f"[emit] n={n} degree={degree} views={views}", flush=True)
    w, h = 96, 64
    t = to_device(_scene(n, degree))
    rng = np.random.default_rng(5)
    cams = [synth.orbit_camera(rng, w, h) for _ in range(views)]
    dL = torch.as_tensor(rng.standard_normal((views, h, w, 3)).astype(np.float32)).cuda()
    base = {k: torch.randn_like(x) for k, x in t.items()}
    single = []
    for v in range(views):
        g = {k: torch.empty_like(x) for k, x in t.items()}
        _backward(t, cams[v:v + 1], dL[v:v + 1].contiguous(), lambda *ws: G.ges_render_backward_views(*ws, g))
        single.append(g)
    grads, more = {k: torch.empty_like(x) for k, x in t.items()}, {k: x.clone() for k, x in base.items()}
    _backward(t, cams, dL, lambda *ws: G.ges_render_backward_views(*ws, grads))
    _backward(t, cams, dL, lambda *ws: G.ges_render_backward_views(*ws, more, accumulate=True))
    for k in t:
        want, onto = single[0][k].clone(), base[k] + single[0][k]
        for g in single[1:]:
            want, onto = want + g[k], onto + g[k]
        assert torch.equal(grads[k], want), k
        assert torch.equal(more[k], onto), k
    assert any(float(x.abs().max()) > 0 for x in grads.values())
    # Adam: two steps fused, against stored gradients and the stand-alone step
    m = {k: 1e-3 * torch.randn_like(x) for k, x in t.items()}
    vv = {k: 1e-6 * torch.rand_like(x) for k, x in t.items()}
    a = [{k: x.clone() for k, x in d.items()} for d in (t, m, vv)]
    b = [{k: x.clone() for k, x in d.items()} for d in (t, m, vv)]
    for step in (7, 8):
        out = {k: torch.empty_like(x) for k, x in t.items()}
        _backward(a[0], cams, dL, lambda *ws: G.ges_render_backward_views_adam(*ws, a[1], a[2], LRS, step, grads=out))
        g = {k: torch.empty_like(x) for k, x in t.items()}
        _backward(b[0], cams, dL, lambda *ws: G.ges_render_backward_views(*ws, g))
        G.ges_adam_step([(b[0][k], g[k], b[1][k], b[2][k], LRS[k]) for k in LRS], step)
        torch.cuda.synchronize()
        for k in t:
            assert torch.equal(out[k], g[k]), k
            for x, y in zip(a, b):
                assert torch.equal(x[k], y[k]), k
