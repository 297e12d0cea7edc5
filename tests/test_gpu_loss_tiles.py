"""SSIM and the frequency mask at the edges of their tiles, against the binary64 oracle.

SSIM: tiles of 64 x 32 pixels of one channel; sizes one below, at and one above a tile.  Tolerances as for the other sizes: |dL| <= 2e-6 + 1e-6 |L| for the mean over all values and 1e-4 of
the largest gradient (the variances divide by C2 ~ 1e-3).
Mask: 5 x 5 pixels make a low pixel, 1,024 of them a segment of the pass across (5,120 pixels), 32 x 16 a tile of the pass
down; four bytes are stored at once where rows start at multiples of 4; more than 512 tiles have their largest taken by
a launch of its own.  Masks are equal wherever the response is not within 1e-4 of the threshold, the binary32 rounding
of a sum of up to 129 x 129 weighted values."""
import numpy as np
import pytest
import torch

from oracle import loss as OL
from oracle import ssim as OS
from paper_2402_10128_amd import ges as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W", [(31, 63), (32, 64), (33, 65), (64, 129), (7, 160), (1, 67), (40, 5)])
def test_ssim_tile_edges(H, W):
    rng = np.random.default_rng(H * 1000 + W)
    tgt = rng.random((H, W, 3)).astype(np.float32)
    img = np.clip(tgt + 0.1 * rng.standard_normal((H, W, 3)), 0, 1).astype(np.float32)
    dl0 = (rng.standard_normal((H, W, 3)) * 1e-3).astype(np.float32)
    loss, dl = torch.tensor(0.25, device="cuda:0"), torch.from_numpy(dl0).cuda()
    G.ges_ssim_loss(torch.from_numpy(img).cuda(), torch.from_numpy(tgt).cuda(), 0.2, loss, dl)
    lref, gref = OS.ssim_loss_and_grad(img, tgt)
    want = 0.25 + 0.2 * lref
    assert abs(float(loss) - want) <= 2e-6 + 1e-6 * abs(want)
    assert np.abs(dl.cpu().numpy() - (dl0 + 0.2 * gref)).max() <= 1e-4 * np.abs(0.2 * gref).max()


@pytest.mark.parametrize("H,W,offset", [(4, 3, 0), (81, 160, 0), (80, 164, 1), (79, 157, 0), (12, 5125, 0), (5001, 1700, 0)])
def test_mask_tile_edges(H, W, offset):
    rng = np.random.default_rng(H + W)
    yy, xx = np.mgrid[0:H, 0:W]
    tgt = (0.5 + 0.4 * np.sin(xx / 19.0)[..., None] * np.cos(yy / 23.0)[..., None]
           + 0.05 * rng.standard_normal((H, W, 3))).astype(np.float32)
    t = torch.from_numpy(tgt).cuda()
    for omega in (0.75, 0.2):
        buf = torch.full((H * W + 8,), 7, dtype=torch.uint8, device="cuda:0")
        scratch = torch.full((G.lib().ges_mask_scratch_bytes(W, H),), 255, dtype=torch.uint8, device="cuda:0")
        mask = buf[offset:offset + H * W]
        assert G.lib().ges_freq_mask(t.data_ptr(), W, H, omega, scratch.data_ptr(), mask.data_ptr(),
                                     torch.cuda.current_stream().cuda_stream) == 0
        got = mask.cpu().numpy().reshape(H, W)
        assert bool((buf[:offset] == 7).all()) and bool((buf[offset + H * W:] == 7).all())
        ref = OL.freq_mask(tgt.astype(np.float64), omega)
        resp = OL.dog_response(tgt.astype(np.float64), omega if omega > 0.5 else omega + 0.5)
        near = (np.abs(resp - 0.5) < 1e-4)[np.arange(H)[:, None] // 5, np.arange(W)[None, :] // 5]
        assert np.array_equal(got[~near], ref[~near]), int((got != ref).sum())


def _mask_over_numbers(tgt, omega):
    """The mask's definition with the largest response taken over those that are numbers; a response that is none
    is not above the threshold."""
    low = OL.downsample(tgt.mean(axis=2))
    om = omega if omega > 0.5 else omega + 0.5
    s2 = 0.1 + 10.0 * om
    with np.errstate(invalid="ignore", divide="ignore"):
        resp = np.abs(OL.blur(low, 2.0 * s2) - OL.blur(low, s2))
        m = resp[~np.isnan(resp)].max(initial=0.0)
        resp = resp / m if m > OL.ZERO_RESPONSE else np.zeros_like(resp)
        bit = (resp > 0.5).astype(np.uint8)
    ys, xs = np.arange(tgt.shape[0])[:, None] // 5, np.arange(tgt.shape[1])[None, :] // 5
    near = np.abs(resp - 0.5) < 1e-4
    return (1 - bit if omega <= 0.5 else bit)[ys, xs], near[ys, xs]


@pytest.mark.parametrize("H,W,patch", [(533, 801, p) for p in ("nan", "minus-nan", "inf", "nan-rows", "all-nan")] +
                         [(5001, 1700, "nan")])
def test_a_mask_with_values_that_are_not_numbers(H, W, patch):
    """A response that is not a number (the pixels within a blur radius of one that is not) takes no part in the
    largest; an infinite one does.  Both sizes: the largest taken by the last kernel's waves, and by a launch of its own."""
    rng = np.random.default_rng(H)
    yy, xx = np.mgrid[0:H, 0:W]
    tgt = (0.5 + 0.4 * np.sin(xx / 19.0)[..., None] * np.cos(yy / 23.0)[..., None]
           + 0.05 * rng.standard_normal((H, W, 3))).astype(np.float32)
    where, value = {"nan": (np.s_[H // 2, W // 3, 1], np.nan), "minus-nan": (np.s_[H // 2, W // 3, 1], -np.nan),
                    "inf": (np.s_[7, 5, 0], np.inf), "nan-rows": (np.s_[:40], np.nan),
                    "all-nan": (np.s_[:], np.nan)}[patch]
    tgt[where] = value
    for omega in (0.75, 0.2):
        ref, near = _mask_over_numbers(tgt.astype(np.float64), omega)
        got = G.ges_freq_mask(torch.from_numpy(tgt).cuda(), omega).cpu().numpy()
        assert np.array_equal(got[~near], ref[~near]), (omega, int((got != ref).sum()))
        if patch in ("nan", "minus-nan", "nan-rows"):
            assert 0 < ref.sum() < ref.size   # the reference: a mask of its own away from them


@pytest.mark.parametrize("scale", [1.0, 2.2e9, 2.7e9])
def test_ssim_of_large_values(scale):
    """Checkerboards whose product of the two denominators, about 3.2 scale^4, lies just below the largest binary32
    number: its reciprocal is subnormal there (a quotient by way of it, without scaling, is 0).  Tolerances as above."""
    H, W = 40, 70
    rng = np.random.default_rng(5)
    board = (np.add(*np.mgrid[0:H, 0:W]) % 2 * 2 - 1)[..., None]
    tgt = (scale * (1 + 0.9 * board + 0.01 * rng.standard_normal((H, W, 3)))).astype(np.float32)
    img = (scale * (1 + 0.8 * board + 0.05 * rng.standard_normal((H, W, 3)))).astype(np.float32)
    loss, dl = torch.zeros((), device="cuda:0"), torch.zeros((H, W, 3), device="cuda:0")
    G.ges_ssim_loss(torch.from_numpy(img).cuda(), torch.from_numpy(tgt).cuda(), 0.2, loss, dl)
    lref, gref = OS.ssim_loss_and_grad(img, tgt)
    assert abs(float(loss) - 0.2 * lref) <= 2e-6 + 1e-6 * 0.2 * lref
    assert np.abs(dl.cpu().numpy() - 0.2 * gref).max() <= 1e-4 * np.abs(0.2 * gref).max()
