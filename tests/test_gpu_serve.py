"""Serving on the GPU: every request of a mixed batch against the oracle (records, per-tile lists and
ranges bit-exact, image within 1e-5 under the flag protocol); a request's image is bit-identical alone, in
a mixed batch and through the plain render path; batched serving beats one-request-at-a-time serving in
throughput and p99 latency."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth
from paper_2402_10128_amd.serve import Server, inspect_arrays, run_stream

from .parity_helpers import IMG_ATOL, image_compare, record_mismatches, to_device

pytestmark = pytest.mark.gpu

RES = [(256, 256), (512, 512), (320, 180), (640, 360)]


def _scenes(sizes, seed=500):
    return [to_device(synth.scene_clusters(n, seed + i).arrays()) for i, n in enumerate(sizes)]


def _requests(n_req, n_scenes, seed=2000):
    return synth.serving_requests(n_req, n_scenes, RES, seed=seed)


def test_served_requests_match_the_oracle():
    """One mixed batch of 8 requests over 3 resident scenes and 4 resolutions (one ragged: 200x136 is 12.5 x
    8.5 tiles): per request, every record bit-exact, the view's key count, every tile's list (its range in
    the batch's sorted ids) equal to the oracle's, and the image within 1e-5 per channel with n_contrib
    equal on unflagged pixels -- every tile of the small views, 48 sampled tiles (random, a 2x2 block and
    the longest lists) of the 1280x720 ones."""
    sizes = [20_000, 50_000, 80_000]
    host = [synth.scene_clusters(n, 500 + i) for i, n in enumerate(sizes)]
    scenes = [to_device(h.arrays()) for h in host]
    plan = [(0, (256, 256)), (1, (200, 136)), (2, (1280, 720)), (0, (512, 512)), (1, (1280, 720)), (2, (200, 136)),
            (1, (256, 256)), (2, (512, 512))]
    reqs = [(k, synth.orbit_camera(np.random.default_rng(3000 + i), w, h)) for i, (k, (w, h)) in enumerate(plan)]
    outs = [torch.zeros((c.height, c.width, 3), device="cuda") for _, c in reqs]
    bufs = [torch.zeros(64 << 20, dtype=torch.uint8, device="cuda") for _ in reqs]
    with Server(4 << 30, max_slots=8) as srv:
        ids = [srv.add_scene(sc) for sc in scenes]
        rids = [srv.submit(ids[k], cam, out, inspect=b) for (k, cam), out, b in zip(reqs, outs, bufs)]
        srv.drain()
        infos = [srv.poll(r) for r in rids]
    assert all(i["state"] == "DONE" for i in infos)
    print("batch sizes:", [i["batch_size"] for i in infos], flush=True)
    assert max(i["batch_size"] for i in infos) > 1
    rng = np.random.default_rng(4)
    for i, ((k, cam), out, buf, info) in enumerate(zip(reqs, outs, bufs, infos)):
        n = sizes[k]
        a = inspect_arrays(buf, n, cam.width, cam.height, info["num_keys"])
        assert "ids" in a, "inspection buffer too small for the batch's sorted ids"
        orc = O.Oracle(host[k].arrays(), host[k].sh_degree, cam, falloff=O.FALLOFF_PHI, tile_cull=O.TILES_ELLIPSE)
        rec = orc.preprocess(O.MODE_F32)
        keys, vals, ranges = orc.build_keys(rec)
        mm = record_mismatches(a["records"], rec)
        assert all(v == 0 for v in mm.values()), (i, mm)
        assert int(a["header"][0]) == len(keys), (i, int(a["header"][0]), len(keys))
        assert int(a["header"][1]) == 0, "error word set"
        g_len = a["ranges"][:, 1].astype(np.int64) - a["ranges"][:, 0]
        o_len = ranges[:, 1] - ranges[:, 0]
        assert np.array_equal(g_len, o_len), i
        assert np.all(a["ranges"][o_len == 0] == 0), "empty tiles must have the range (0, 0)"
        for t in np.nonzero(o_len)[0]:
            g0, g1 = a["ranges"][t]
            assert np.array_equal(a["ids"][g0:g1], vals[ranges[t, 0]:ranges[t, 1]]), (i, t)
        T = orc.TX * orc.TY
        if cam.width * cam.height > 512 * 512:
            block = [ty * orc.TX + tx for ty in (20, 21) for tx in (38, 39)]
            longest = list(np.argsort(o_len)[-4:])
            tiles = np.unique(np.concatenate([rng.choice(T, 40, replace=False), block, longest])).astype(np.int32)
        else:
            tiles = None
        ref = orc.render(rec, vals, ranges, tiles=tiles)
        mask = np.zeros((cam.height, cam.width), bool)
        for t in (range(T) if tiles is None else tiles):
            ty, tx = divmod(int(t), orc.TX)
            mask[16 * ty:16 * ty + 16, 16 * tx:16 * tx + 16] = True
        cmp = image_compare(out.cpu().numpy(), ref, pixels_mask=mask)
        print(f"  request {i}: scene {k} {cam.width}x{cam.height} K={len(keys)} batch {info['batch_size']} "
              f"tiles {'all' if tiles is None else len(tiles)} image {cmp}", flush=True)
        assert cmp["max_err"] <= IMG_ATOL and cmp["flagged_max_err"] <= IMG_ATOL, (i, cmp)
        unf = mask & ~ref["flags"].astype(bool)
        assert np.array_equal(a["n_contrib"][unf], ref["n_contrib"][unf].astype(np.uint32)), i


def test_alone_equals_mixed_equals_plain_render():
    scenes = _scenes([20_000, 50_000, 80_000])
    reqs = _requests(12, len(scenes))
    outs_mixed = [torch.zeros((c.height, c.width, 3), device="cuda") for _, c in reqs]
    outs_alone = [torch.zeros_like(o) for o in outs_mixed]
    with Server(4 << 30, max_slots=8) as s:
        ids = [s.add_scene(sc) for sc in scenes]
        # mixed: everything at once (batched)
        rids = [s.submit(ids[k], cam, out) for (k, cam), out in zip(reqs, outs_mixed)]
        s.drain()
        sizes = [s.poll(r)["batch_size"] for r in rids]
        assert all(s.poll(r)["state"] == "DONE" for r in rids)
        # alone: one at a time
        for (k, cam), out in zip(reqs, outs_alone):
            r = s.submit(ids[k], cam, out)
            s.drain()
            assert s.poll(r)["batch_size"] == 1
    print("batch sizes in the mix:", sizes)
    assert max(sizes) > 1
    for a, b in zip(outs_alone, outs_mixed):
        assert torch.equal(a, b)
    # and equal to the plain render path (same kernels, single view)
    for (k, cam), out in zip(reqs[:4], outs_alone[:4]):
        img, _ = G.render(scenes[k], cam, tile_cull=G.TILES_ELLIPSE)
        assert torch.equal(img, out)


@pytest.mark.parametrize("slots", [1, 8])
def test_requests_behind_one_whose_keys_do_not_fit(slots):
    """A pool with room for a large request's workspace but not for its keys: that request fails with OUT_OF_MEMORY
    while its sort may still be running, and the images of the requests queued behind it, which get the same bytes of the pool
    on the other stream, are those of the plain render bit for bit."""
    n = 1_000_000
    large = synth.scene_clusters(n, 520).arrays()
    large["log_scales"] += np.float32(1.5)
    large, small = to_device(large), _scenes([2_000])[0]
    cam = synth.orbit_camera(np.random.default_rng(5), 1280, 720)
    cams = [synth.orbit_camera(np.random.default_rng(6 + i), 256, 256) for i in range(6)]
    pool = G.ges_workspace_query(n, 1280, 720)[0] + (16 << 20)
    outs = [torch.zeros((256, 256, 3), device="cuda") for _ in cams]
    big = torch.zeros((720, 1280, 3), device="cuda")
    want = [G.render(small, c, tile_cull=G.TILES_ELLIPSE)[0] for c in cams]
    torch.cuda.synchronize()
    with Server(pool, max_slots=slots) as s:
        a, b = s.add_scene(large), s.add_scene(small)
        for _ in range(3):
            first = s.submit(a, cam, big)
            rids = [s.submit(b, c, o) for c, o in zip(cams, outs)]
            s.drain()
            info = s.poll(first)
            assert info["state"] == "FAILED" and info["status"] == 3, info
            assert all(s.poll(r)["state"] == "DONE" for r in rids)
            for o, w in zip(outs, want):
                assert torch.equal(o, w)
                o.zero_()


def test_batched_beats_sequential_throughput_and_p99():
    scenes = _scenes([200_000, 500_000, 1_000_000])
    reqs = _requests(48, len(scenes), seed=2100)
    outs = [torch.zeros((c.height, c.width, 3), device="cuda") for _, c in reqs]
    results = {}
    for mode in ("sequential", "batched"):
        with Server(16 << 30, max_slots=16, sequential=(mode == "sequential")) as s:
            ids = [s.add_scene(sc) for sc in scenes]
            rq = [(ids[k], cam) for k, cam in reqs]
            run_stream(s, rq[:8], outs[:8], None)          # warm-up
            results[mode] = run_stream(s, rq, outs, None)
    seq, bat = results["sequential"], results["batched"]
    print(f"sequential: {seq['mpix_s']:.1f} Mpix/s p50 {seq['p50_ms']:.2f} p99 {seq['p99_ms']:.2f}")
    print(f"batched:    {bat['mpix_s']:.1f} Mpix/s p50 {bat['p50_ms']:.2f} p99 {bat['p99_ms']:.2f} "
          f"mean batch {bat['mean_batch']:.1f}")
    assert seq["all_done"] and bat["all_done"]
    assert bat["mpix_s"] > seq["mpix_s"]
    assert bat["p99_ms"] < seq["p99_ms"]
