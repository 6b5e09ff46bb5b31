"""The two-column detector walk on frames whose float32 bounds stay open in most
rows, so that its strips change over to exact responses: from the first rows,
in the middle of a strip, at the frame's edges and inside, for each strip
height (a flat frame in the same call makes up the pixels), against the
oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [(40, 40), (124, 100), (253, 70), (400, 139), (517, 200)]


def image(kind, w, h, rng):
    y, x = np.mgrid[0:h, 0:w]
    if kind == "dots":
        return np.where(rng.random((h, w)) < 0.1, 255, 0).astype(np.uint8)
    if kind == "ramps":                        # straight edges: responses near 0 beside large traces
        return ((x * 7 + (y // 9) * 31) % 256).astype(np.uint8)
    noise = rng.integers(0, 256, (h, w), dtype=np.uint8)
    checks = np.where(((x // 2) + (y // 2)) % 2, 255, 0).astype(np.uint8)
    return np.where(y % 64 < 20, noise, checks)


@pytest.mark.parametrize("filler", [0, 1 << 20, 3 << 20, 14 << 20])
@pytest.mark.parametrize("kind", ["dots", "ramps", "turns"])
@pytest.mark.parametrize("pad,shift,border,quality", [(0, 0, 0, 0.0), (3, 1, 2, 0.02), (12, 4, 5, 1.0)])
def test_exact_walk(kind, filler, pad, shift, border, quality):
    import torch
    from paper_2607_01757_amd import lk

    print(kind, filler, pad, shift, border, quality, flush=True)
    rng = np.random.default_rng(11)
    frames, want, corners = [], [], 3000
    for w, h in SIZES:
        im = image(kind, w, h, rng)
        want.append(np.asarray(oracle.gftt(im, r=1, quality=quality, min_dist=3, max_corners=corners, border=border)).reshape(-1, 2))
        store = torch.zeros((shift + h * (w + pad),), dtype=torch.uint8)
        torch.as_strided(store, (h, w), (w + pad, 1), shift).copy_(torch.from_numpy(im))
        frames.append({"img": torch.as_strided(store.cuda(), (h, w), (w + pad, 1), shift),
                       "out_xy": torch.full((corners, 2), -1.0, device="cuda"),
                       "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")})
    if filler:
        frames.append({"img": torch.full((1024, filler // 1024), 9, dtype=torch.uint8, device="cuda"),
                       "out_xy": torch.empty((corners, 2), device="cuda"),
                       "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")})
    ctx = lk.lk_context_create(0, 0)
    try:
        det = lk.lk_detector_create(ctx, len(frames), sum(f["img"].numel() for f in frames))
        lk.lk_detect_corners(det, frames, lk.gftt_params(1, 3, corners, border, quality))
        torch.cuda.synchronize()
        for size, f, xy in zip(SIZES, frames, want):
            got = f["out_xy"][:int(f["count"].item())].cpu().numpy()
            assert np.array_equal(got, xy), size
        lk.lk_detector_destroy(det)
    finally:
        lk.lk_context_destroy(ctx)
