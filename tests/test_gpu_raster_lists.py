"""Raster passes at the edges of their list walks: lists of one splat, around the groups a wave takes at a time,
around one and two staged batches, and through several list segments, on a frame whose tiles are ragged in both
directions; against the oracle with the parity tolerances (parity_helpers).  And a splat whose colour is not
finite: it may only reach the pixels that composite it."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2402_10128_amd import synth

from .parity_helpers import (IMG_ATOL, assert_grad_ok, gpu_render, grad2d_check, grad3d_check, image_compare,
                             oracle_full)

pytestmark = pytest.mark.gpu
W, H = 23, 19


def _scene(n, seed, logit, log_scale):
    sc = synth.scene_uniform(n, seed).arrays()
    rng = np.random.default_rng(seed + 1)
    sc["opacity_logits"] = rng.normal(logit, 0.3, n).astype(np.float32)
    sc["log_scales"] = rng.normal(log_scale, 0.4, (n, 3)).astype(np.float32)
    return sc, synth.pinhole(W, H, (0.0, 0.0, -4.0), fov_x_deg=40.0)


# thin opacities, so that the walk reaches the end of the list; wide splats, so that every tile lists them
LENGTHS = [1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 257, 700]


@pytest.mark.parametrize("falloff", [O.FALLOFF_PHI, O.FALLOFF_GEF], ids=["phi", "gef"])
@pytest.mark.parametrize("n", LENGTHS)
def test_list_lengths_against_the_oracle(n, falloff):
    print(f"[lists] n={n} falloff={falloff}", flush=True)
    sc, cam = _scene(n, 40 + n, -4.0 if n > 200 else -3.0, -1.5)
    dL = np.random.default_rng(n).standard_normal((H, W, 3)).astype(np.float32)
    gpu = gpu_render(sc, 0, cam, falloff, O.TILES_ELLIPSE, bg=(0.1, 0.2, 0.3), dL=dL)
    ref = oracle_full(sc, 0, cam, falloff, O.TILES_ELLIPSE, bg=(0.1, 0.2, 0.3), dL=dL.astype(np.float64))
    assert np.array_equal(gpu["sorted_ids"], ref["values"])
    cmp = image_compare(gpu["img"], ref["out"])
    assert cmp["max_err"] <= IMG_ATOL and cmp["flagged_max_err"] <= IMG_ATOL, cmp
    fl = ref["out"]["flags"].astype(bool)
    assert np.array_equal(gpu["n_contrib"][~fl], ref["out"]["n_contrib"][~fl].astype(np.uint32))
    assert_grad_ok("2-D", grad2d_check(gpu["grad2d"][:, :10], ref["g2d"], ref["delta"], ref["mass"], ref["ebound"]))
    for k in gpu["grads"]:
        assert_grad_ok(f"d{k}", grad3d_check(gpu["grads"][k], ref["grads"][k], ref["allow"][k]))


@pytest.mark.parametrize("odd", [0, 1, 64, 150], ids=lambda k: f"splat{k}")
def test_a_colour_that_is_not_finite_stays_on_its_pixels(odd):
    """SH of degree 1 near the largest binary32 number gives an infinite colour.  Every pixel that does not
    composite that splat is the pixel of the scene with an ordinary colour in its place, bit for bit."""
    n = 200
    base, _ = _scene(n, 9, -2.0, -3.0)
    eye = np.float32([-2.3, -2.3, -2.3])   # diagonal view: the three degree-1 terms add up past the largest number
    cam = synth.pinhole(W, H, tuple(eye), fov_x_deg=40.0)
    sh = np.zeros((n, 4, 3), np.float32)
    sh[:, :1] = base["sh"]
    plain = dict(base, sh=sh)
    far = base["means"][odd] - eye
    wild = dict(base, sh=sh.copy())
    wild["sh"][odd, 0] = 3e38
    for k, c in ((1, -far[1]), (2, far[2]), (3, -far[0])):
        wild["sh"][odd, k] = np.sign(c) * np.float32(3.4e38)
    print(f"[colour] splat {odd}", flush=True)
    a = gpu_render(plain, 1, cam, 0, O.TILES_SQUARE)
    b = gpu_render(wild, 1, cam, 0, O.TILES_SQUARE)
    finite = np.isfinite(b["img"]).all(axis=2)
    assert np.isinf(b["records"][odd, 8:11]).all()
    assert (~finite).any() and finite.any()
    assert np.array_equal(a["img"][finite], b["img"][finite])
    assert np.array_equal(a["n_contrib"], b["n_contrib"]) and np.array_equal(a["final_T"], b["final_T"])


def test_gradients_around_a_colour_that_is_not_finite():
    """Lists of several segments of the backward's walk, with one splat of infinite colour far back in them.  A splat
    further front, in another segment of every list the two share, that takes no pixel the infinite one takes has the
    gradients of the scene with an ordinary colour in its place."""
    n = 1500
    base, _ = _scene(n, 9, -3.0, -3.2)
    eye = np.float32([-2.3, -2.3, -2.3])   # as above
    cam = synth.pinhole(W, H, tuple(eye), fov_x_deg=40.0)
    sh = np.zeros((n, 4, 3), np.float32)
    sh[:, :1] = base["sh"]
    plain = dict(base, sh=sh)
    dL = np.random.default_rng(4).standard_normal((H, W, 3)).astype(np.float32)
    a = gpu_render(plain, 1, cam, 0, O.TILES_SQUARE, dL=dL)
    rec, tx = a["records"], (W + 15) // 16
    lists = [list(a["sorted_ids"][r0:r1]) for r0, r1 in a["ranges"]]

    def footprint(i, slack):
        dx, dy = rec[i, 0] - np.arange(W)[None, :], rec[i, 1] - np.arange(H)[:, None]
        return rec[i, 2] * dx * dx + 2 * rec[i, 3] * dx * dy + rec[i, 4] * dy * dy <= rec[i, 5] * slack

    # the last splat of the longest list that a pixel composites, with a footprint of a few pixels
    t = int(np.argmax([len(l) for l in lists]))
    y0, x0 = 16 * (t // tx), 16 * (t % tx)
    last = int(a["n_contrib"][y0:y0 + 16, x0:x0 + 16].max())
    assert last > 3 * 64
    odd = next(int(i) for i in reversed(lists[t][:last]) if 0 < footprint(i, 1.0)[y0:y0 + 16, x0:x0 + 16].sum() <= 60)
    far = base["means"][odd] - eye
    wild = dict(base, sh=sh.copy())
    wild["sh"][odd, 0] = 3e38
    for k, c in ((1, -far[1]), (2, far[2]), (3, -far[0])):
        wild["sh"][odd, k] = np.sign(c) * np.float32(3.4e38)
    b = gpu_render(wild, 1, cam, 0, O.TILES_SQUARE, dL=dL)
    assert np.isinf(b["records"][odd, 8:11]).all()
    pixels = ~np.isfinite(b["img"]).all(axis=2)
    assert pixels.any()
    checked = 0
    for i in range(n):
        shared = [l for l in lists if i in l and odd in l]
        if i == odd or not shared or any(l.index(i) // 64 >= l.index(odd) // 64 for l in shared):
            continue
        if (footprint(i, 1.001) & pixels).any():
            continue
        for k in a["grads"]:
            assert np.array_equal(a["grads"][k][i], b["grads"][k][i]), (i, k)
        checked += 1
    print(f"[colour] {checked} splats in front, {int(pixels.sum())} pixels take the infinite one", flush=True)
    assert checked > 20
