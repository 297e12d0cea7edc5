"""The sum of the backward's rows by splat: ranges of 8 words of marks (256 slots) per wave up to 2^25 slots, of 32 beyond,
and chunks of 64 rows with few runs (up to 12: a component per lane) or many (a run per lane).

All add a splat's rows in slot order in binary64, so a frame whose key workspace has room for more than 2^25 slots
gives the bits of one with just its own; that those are right is what the comparisons with the oracle elsewhere
say."""
import numpy as np
import pytest
import torch

from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

from .parity_helpers import to_device

pytestmark = pytest.mark.gpu


def _gradients(arrays, cam, dL, capacity):
    t = to_device(arrays)
    s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
    c, p = G.camera_struct(cam), G.params_struct(0, G.TILES_ELLIPSE)
    frame = G.Frame.create(s.n, c.width, c.height)
    k = G.ges_preprocess(s, c, p, frame.splat_ws, True)
    frame.ensure_keys(max(k, capacity))
    out = torch.empty((c.height, c.width, 3), device="cuda")
    G.ges_render_forward(s, c, p, frame.splat_ws, frame.key_ws, frame.num_keys, frame.pixel_ws, out)
    grads = {n: torch.zeros_like(t[n]) for n in G.SPLAT_PARAMS}
    G.ges_render_backward(s, c, p, frame.splat_ws, frame.key_ws, frame.pixel_ws, dL, grads)
    return k, {n: g.cpu().numpy() for n, g in grads.items()}


@pytest.mark.parametrize("sizes", ["tiny", "screen", "mixed"])
def test_ranges_and_runs(sizes):
    n = {"tiny": 20000, "screen": 30, "mixed": 3000}[sizes]
    sc = synth.scene_uniform(n, 77)
    if sizes == "tiny":
        sc.log_scales[:] = -6.0            # a row or two each: up to 64 runs in 64 rows
    elif sizes == "screen":
        sc.log_scales[:] = 1.5             # every tile of the frame (1,938): one splat's rows go through many ranges
        sc.opacity_logits[:] = -3.0
    else:
        sc.log_scales[:] = np.random.default_rng(5).choice([-6.0, -3.0, -1.0], (n, 1)).astype(np.float32)
        sc.opacity_logits[:] = -2.0
    cam = synth.pinhole(816, 600, (0.0, 0.0, -4.0))
    dL = torch.randn((600, 816, 3), generator=torch.Generator().manual_seed(1)).cuda()
    k, a = _gradients(sc.arrays(), cam, dL, 0)
    _, b = _gradients(sc.arrays(), cam, dL, 2**25 + 1)
    assert k < 2**25 and any(np.abs(g).max() > 0 for g in a.values())
    for name in a:
        assert np.array_equal(a[name], b[name]), name
