"""Which walks of the backward raster are cut is decided on the device by their lengths, for frames of up to 6,144 tiles.
A frame at that limit with even walks (not cut) and with all splats in one dense cluster (cut): its 2-D gradients are those
of the same frame as one of two views, which have more tiles and are never cut, bit for bit."""
import numpy as np
import pytest
import torch

from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

pytestmark = pytest.mark.gpu
W, H, N = 1536, 1024, 150_000   # 6,144 tiles


def _grad2d(scene, cam, views, falloff, dL):
    s, c = G.splats_struct(*(scene[k] for k in G.SPLAT_PARAMS)), [G.camera_struct(cam)] * views
    p = G.params_struct(falloff, G.TILES_ELLIPSE, 0.1, (0.1, 0.2, 0.3), flags=G.RASTER_KEEP_GRAD2D)
    f = G.Frame.create(N, W, H, views=views)
    f.ensure_keys(G.ges_preprocess_views(s, c, p, f.splat_ws, True))
    img = torch.empty((views, H, W, 3), device="cuda")
    G.ges_render_forward_views(s, c, p, f.splat_ws, f.key_ws, f.num_keys, f.pixel_ws, img)
    grads = {k: torch.empty_like(scene[k]) for k in G.SPLAT_PARAMS}
    G.ges_render_backward_views(s, c, p, f.splat_ws, f.key_ws, f.pixel_ws, dL.expand(views, H, W, 3).contiguous(), grads)
    a = G.frame_arrays(f, N)
    return a["grad2d"][:, :10], a["tile_work"].astype(np.int64)


@pytest.mark.parametrize("falloff", [0, 1], ids=["phi", "gef"])
@pytest.mark.parametrize("spread,cut", [(1.0, False), (0.05, True)], ids=["even", "dense"])
def test_gradients_do_not_depend_on_the_cut(spread, cut, falloff):
    scene = synth.scene_clusters_device(N, 5, torch.device("cuda"), degree=0)
    scene["means"].mul_(spread)
    if cut:
        scene["beta"].fill_(2.0)   # the tails of smaller powers would reach every tile
    cam = synth.orbit_camera(np.random.default_rng(6), W, H)
    dL = torch.randn((1, H, W, 3), generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
    one, work = _grad2d(scene, cam, 1, falloff, dL)
    two, _ = _grad2d(scene, cam, 2, falloff, dL)
    print(f"[cut] spread {spread} falloff {falloff} longest {work.max()} of {work.sum()}", flush=True)
    assert (work.max() * 926 > work.sum()) == cut   # the case is on the side of the rule it stands for
    assert np.any(one != 0) and np.array_equal(one, two)
