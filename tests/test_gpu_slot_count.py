"""The slot count that ges_preprocess hands to the host while the depth sort goes on."""
import pytest
import torch

from paper_2402_10128_amd import ges as G
from paper_2402_10128_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5_000, 2_000_000], ids=["one-block", "radix"])
def test_nothing_runs_in_the_workspace_after_a_count_that_is_too_large(n):
    """Splats that cover all 2^20 tiles of a 16384 x 16384 frame: the count exceeds 2^32 - 2, and when the call has
    failed with CAPACITY its stream is idle (with the second size the sort takes some tens of microseconds)."""
    W = H = 16384
    g = torch.Generator(device="cuda").manual_seed(3)
    rand = lambda *s: torch.rand(s, generator=g, device="cuda")
    scene = dict(means=rand(n, 3) - 0.5, log_scales=torch.full((n, 3), 6.0, device="cuda"),
                 quats=rand(n, 4) + 0.1, opacity_logits=torch.full((n,), 2.0, device="cuda"), sh=rand(n, 1, 3),
                 beta=torch.full((n,), 2.0, device="cuda"))
    s = G.splats_struct(*(scene[k] for k in G.SPLAT_PARAMS))
    c, p = G.camera_struct(synth.pinhole(W, H, (0.0, 0.0, -4.0))), G.params_struct()
    ws = torch.empty(G.ges_workspace_query(n, W, H)[0], dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    for _ in range(3):
        print(f"[slot count] {n} splats", flush=True)
        with pytest.raises(G.GESError) as e:
            G.ges_preprocess(s, c, p, ws, True)
        idle = torch.cuda.current_stream().query()
        assert e.value.status == 2 and idle


def test_a_workspace_dropped_after_the_count_is_not_handed_out_while_the_sort_runs():
    """The count of 2M splats on a side stream, given or made the current one, then the workspace (allocated for another) is
    dropped without a render: as long as the side stream works, an allocation of its size gets other memory."""
    n, W, H = 2_000_000, 256, 256
    scene = synth.scene_clusters_device(n, 3, torch.device("cuda"), degree=0)
    s = G.splats_struct(*(scene[k] for k in G.SPLAT_PARAMS))
    c, p = G.camera_struct(synth.pinhole(W, H, (0.0, 0.0, -8.0))), G.params_struct()
    size = G.ges_workspace_query(n, W, H)[0]
    side = torch.cuda.Stream()
    busy = 0
    for k in range(20):
        ws = torch.empty(size, dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        if k % 3 == 0:
            G.ges_preprocess_views(s, [c], p, ws, True, stream=side)
        elif k % 3 == 1:
            G.ges_preprocess(s, c, p, ws, True, stream=side)
        else:
            with torch.cuda.stream(side):
                G.ges_preprocess(s, c, p, ws, True)
        at = ws.data_ptr()
        del ws
        other = torch.empty(size, dtype=torch.uint8, device="cuda")
        if not side.query():
            busy += 1
            assert other.data_ptr() != at
        del other
        torch.cuda.synchronize()
    print(f"[slot count] {busy} of 20 drops while the side stream worked", flush=True)
    assert busy > 0
