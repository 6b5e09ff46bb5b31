"""The detector's selection windows against the oracle, where their sort, their
ends and their chunks can go wrong: many equal responses (one step of the
counting sort holds them all), a few equal ones among distinct ones, windows
that end inside a bucket, more unblocked candidates than one chunk decides, and
corners taken before the next window."""
import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def dots(h, w, step, seed=None):
    """Equal small squares on a lattice (equal responses), on noise of +-1
    with a seed (distinct ones)."""
    im = np.full((h, w), 60, np.int32)
    for y in range(8, h - 8, step):
        for x in range(8, w - 8, step):
            im[y:y + 3, x:x + 3] = 200
    if seed is not None:
        im += np.random.default_rng(seed).integers(-1, 2, im.shape)
    return im.astype(np.uint8)


IMAGES = {
    "lattice 7": lambda: dots(301, 405, 7),
    "lattice 16": lambda: dots(480, 640, 16),
    "noisy lattice": lambda: dots(301, 405, 7, 1),
    "noise": lambda: np.random.default_rng(2).integers(0, 256, (200, 333), dtype=np.uint8),
    "texture": lambda: synth.pair(3, 640, 480, 8).next,
}


@pytest.mark.parametrize("name", IMAGES)
@pytest.mark.parametrize("min_dist,corners,quality,n_occ", [
    (0, 700, 0.01, 0), (2, 4096, 0.0, 0), (5, 600, 0.01, 0), (12, 1500, 0.001, 40), (30, 200, 0.01, 0), (90, 50, 0.05, 3)])
def test_windows(name, min_dist, corners, quality, n_occ):
    import torch
    from paper_2607_01757_amd import lk

    im = IMAGES[name]()
    h, w = im.shape
    occ = np.random.default_rng(5).uniform([0, 0], [w, h], (n_occ, 2)).astype(np.float32)
    want = np.asarray(oracle.gftt(im, r=1, quality=quality, min_dist=min_dist, max_corners=corners, border=4,
                                  occupied=occ if n_occ else None)).reshape(-1, 2)
    ctx = lk.lk_context_create(0, 0)
    try:
        det = lk.lk_detector_create(ctx, 1, w * h)
        f = {"img": torch.from_numpy(im).cuda(), "out_xy": torch.full((corners, 2), -1.0, device="cuda"),
             "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")}
        if n_occ:
            f["occupied"] = torch.from_numpy(occ).cuda()
        lk.lk_detect_corners(det, [f], lk.gftt_params(1, min_dist, corners, 4, quality))
        torch.cuda.synchronize()
        got = f["out_xy"][:int(f["count"].item())].cpu().numpy()
        assert np.array_equal(got, want)
        lk.lk_detector_destroy(det)
    finally:
        lk.lk_context_destroy(ctx)
