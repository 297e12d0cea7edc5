"""The binning's radix passes by the size of their blocks: up to 2^21 items, beyond, and beyond 2^26 (items and slots);
and its chunk offsets, added up by the duplication up to 2^19 items and scanned beyond.

The order is checked on the device, where the sorted lists are: pairs ascend by tile and, within a tile, by candidate
slot (the passes are stable and slots follow the depth order); every slot occurs once; along the slots the
splats' depths ascend.  Depths are binary32 values of about 3 to 5, so two splats whose z differ by less than an
ulp (4.8e-7) may stand in either order."""
import pytest
import torch

from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,log_scale", [(2**19, -9.0), (2**19 + 1, -9.0), (2**21, -9.0), (2**21 + 1, -9.0),
                                         (400_000, -2.45), (2**26 + 1, -12.0)],
                         ids=["512k", "512k+1", "2M", "2M+1", "slots>64M", "64M+1"])
def test_lists_of_large_scenes(n, log_scale):
    print(f"[large sort] n={n}", flush=True)
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev).manual_seed(n)
    means = torch.rand((n, 3), generator=g, device=dev) * 2 - 1
    t = dict(means=means, log_scales=torch.full((n, 3), log_scale, device=dev),
             quats=torch.tensor([1.0, 0, 0, 0], device=dev).repeat(n, 1),
             opacity_logits=torch.ones(n, device=dev), sh=torch.rand((n, 1, 3), generator=g, device=dev),
             beta=torch.full((n,), 2.0, device=dev))
    s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
    cam = synth.pinhole(1600, 1040, (0.0, 0.0, -4.0))
    c, p = G.camera_struct(cam), G.params_struct(0, G.TILES_SQUARE)
    frame = G.Frame.create(n, c.width, c.height)
    k = G.ges_preprocess(s, c, p, frame.splat_ws, True)
    frame.ensure_keys(k)
    if log_scale > -9:
        assert 2**26 < k < 2**28
    out = torch.empty((c.height, c.width, 3), device=dev)
    G.ges_render_forward(s, c, p, frame.splat_ws, frame.key_ws, k, frame.pixel_ws, out)
    v = frame.view(0)

    def part(ptr, nbytes, ws):
        return ws[ptr - ws.data_ptr():][:nbytes]

    keys = int(part(v.stats, 8, frame.splat_ws).view(torch.int64))
    assert keys == k > n // 2   # square tiles: every candidate is a pair
    tiles = part(v.sorted_tiles, 4 * k, frame.key_ws).view(torch.int32)
    pairs = part(v.sorted_pairs, 8 * k, frame.key_ws).view(torch.int32).reshape(k, 2)
    ids, slots = pairs[:, 0], pairs[:, 1]
    assert bool(((tiles[1:] > tiles[:-1]) | ((tiles[1:] == tiles[:-1]) & (slots[1:] > slots[:-1]))).all())
    by_slot = torch.full((k,), -1, dtype=torch.int32, device=dev)
    by_slot[slots.long()] = ids
    assert int(by_slot.min()) >= 0   # k slots below k, none twice
    z = means[by_slot.long(), 2]
    assert float((z[1:] - z[:-1]).min()) >= -1e-6
    ranges = part(v.tile_ranges, 8 * v.tiles_x * v.tiles_y, frame.splat_ws).view(torch.int32).reshape(-1, 2).long()
    counts = torch.bincount(tiles, minlength=v.tiles_x * v.tiles_y)
    ends = counts.cumsum(0)
    assert torch.equal(ranges[counts > 0], torch.stack([ends - counts, ends], 1)[counts > 0])
