"""The binning's one-block sorts and scans at the edges of their range (one item, a wave, a round of the block, the
largest they take and one more), against the oracle's lists; and the slot count handed to the host while the sort
runs: from several threads at once, for no splat, and under capture, where it stays refused."""
import threading

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

from .parity_helpers import to_device

pytestmark = pytest.mark.gpu


def _lists(arrays, cam, cull):
    t = to_device(arrays)
    s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
    c, p = G.camera_struct(cam), G.params_struct(0, cull)
    frame = G.Frame.create(s.n, c.width, c.height)
    k = G.ges_preprocess(s, c, p, frame.splat_ws, True)
    frame.ensure_keys(k)
    out = torch.empty((c.height, c.width, 3), device="cuda")
    G.ges_render_forward(s, c, p, frame.splat_ws, frame.key_ws, k, frame.pixel_ws, out)
    torch.cuda.synchronize()
    return k, G.frame_arrays(frame, s.n)


@pytest.mark.parametrize("size", [(16, 16), (200, 136), (400, 300)], ids=["1_tile", "117_tiles", "475_tiles"])
@pytest.mark.parametrize("n", [1, 63, 65, 1024, 1025, 8192, 8193])
def test_lists_of_small_scenes(n, size):
    """8,192 items or slots are one block's work; 8,193 take the general path."""
    w, h = size
    print(f"[small sort] n={n} {w}x{h}", flush=True)
    sc = synth.scene_uniform(n, 500 + n)
    sc.log_scales -= np.float32(1.0)   # few tiles per splat, so that the slots cross the edge with the items
    sc.means[n // 2:] = sc.means[: n - n // 2]   # equal depths: the index decides
    cam = synth.pinhole(w, h, (0.0, 0.0, -4.0))
    k, a = _lists(sc.arrays(), cam, G.TILES_ELLIPSE)
    orc = O.Oracle(sc.arrays(), 0, cam, falloff=O.FALLOFF_PHI, tile_cull=O.TILES_ELLIPSE)
    rec = orc.preprocess(O.MODE_F32)
    keys, vals, ranges = orc.build_keys(rec)
    assert a["keys"] == len(keys) <= k
    assert np.array_equal(a["sorted_tiles"].astype(np.uint64), keys >> np.uint64(32))
    assert np.array_equal(a["sorted_ids"], vals) and np.array_equal(a["ranges"].astype(np.int64), ranges)
    assert len(np.unique(a["sorted_slots"])) == len(keys)


def test_no_splat_and_all_culled():
    cam = synth.pinhole(40, 24, (0.0, 0.0, -4.0))
    for n in (0, 50, 9000):
        sc = synth.scene_uniform(max(n, 1), 3).arrays()
        sc = {k: v[:n] for k, v in sc.items()}
        sc["means"] = sc["means"] + np.float32([0, 0, -50])   # behind the camera
        k, a = _lists(sc, cam, G.TILES_SQUARE)
        assert k == 0 and a["keys"] == 0 and not a["ranges"].any()


def test_slot_counts_from_several_threads():
    """Calls on their own streams and workspaces at once: each gets its own count."""
    jobs = []
    for j, n in enumerate([500, 3000, 9000, 30000, 700, 20000]):
        t = to_device(synth.scene_clusters(n, 60 + j).arrays())
        s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
        c = G.camera_struct(synth.orbit_camera(np.random.default_rng(j), 320, 200))
        jobs.append((t, s, c, G.Frame.create(s.n, 320, 200), torch.cuda.Stream()))
    p = G.params_struct(0, G.TILES_ELLIPSE)
    want = [G.ges_preprocess(s, c, p, f.splat_ws, True) for _, s, c, f, _ in jobs]
    torch.cuda.synchronize()
    got = [set() for _ in jobs]

    def work(j):
        _, s, c, f, stream = jobs[j]
        for _ in range(20):
            got[j].add(G.ges_preprocess(s, c, p, f.splat_ws, True, stream))

    threads = [threading.Thread(target=work, args=(j,)) for j in range(len(jobs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert [g == {w} for g, w in zip(got, want)] == [True] * len(jobs), (got, want)


def test_reading_the_count_under_capture_is_refused():
    t = to_device(synth.scene_uniform(100, 1).arrays())
    s = G.splats_struct(*(t[k] for k in G.SPLAT_PARAMS))
    c, p = G.camera_struct(synth.pinhole(32, 32, (0.0, 0.0, -4.0))), G.params_struct()
    f = G.Frame.create(s.n, 32, 32)
    k = G.ges_preprocess(s, c, p, f.splat_ws, True)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(G.GESError):
            G.ges_preprocess(s, c, p, f.splat_ws, True)
        torch.zeros(1, device="cuda")
    assert G.ges_preprocess(s, c, p, f.splat_ws, True) == k
