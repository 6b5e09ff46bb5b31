"""The two-column detector walk (block radius 1, no response map) against the
oracle where it can go wrong: widths and heights around its strips, rows and
frames that are not 4-byte aligned, equal responses that its float32 bounds
cannot tell apart, borders, quality 0, and each strip height (chosen by the
pixels of the call: a flat frame in the same call makes them up)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [(3, 3), (4, 5), (5, 64), (61, 9), (122, 8), (123, 17), (124, 33), (125, 7), (131, 40), (247, 16), (248, 65),
         (249, 31), (260, 130), (387, 66)]


def image(kind, w, h, rng):
    if kind == "noise":
        return rng.integers(0, 256, (h, w), dtype=np.uint8)
    if kind == "near-flat":                    # small responses, many of them equal
        return (100 + rng.integers(0, 2, (h, w))).astype(np.uint8)
    y, x = np.mgrid[0:h, 0:w]                  # a pattern that repeats: equal responses everywhere
    return np.where(((x // 3) + (y // 3)) % 2, 255, 0).astype(np.uint8)


@pytest.mark.parametrize("filler", [0, 1 << 20, 3 << 20, 14 << 20])
@pytest.mark.parametrize("kind", ["noise", "near-flat", "checks"])
@pytest.mark.parametrize("pad,shift,border,quality", [(0, 0, 0, 0.0), (1, 1, 3, 0.01), (4, 4, 1, 0.3), (3, 0, 8, 1.0)])
def test_pairs(kind, filler, pad, shift, border, quality):
    import torch
    from paper_2607_01757_amd import lk

    print(kind, filler, pad, shift, border, quality, flush=True)
    rng = np.random.default_rng(7)
    frames, want, corners = [], [], 600
    for w, h in SIZES:
        im = image(kind, w, h, rng)
        want.append(np.asarray(oracle.gftt(im, r=1, quality=quality, min_dist=0, max_corners=corners, border=border)).reshape(-1, 2))
        store = torch.full((shift + h * (w + pad),), 77, dtype=torch.uint8)
        view = torch.as_strided(store, (h, w), (w + pad, 1), shift)
        view.copy_(torch.from_numpy(im))
        dev = torch.as_strided(store.cuda(), (h, w), (w + pad, 1), shift)
        frames.append({"img": dev, "out_xy": torch.full((corners, 2), -1.0, device="cuda"),
                       "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")})
    if filler:
        frames.append({"img": torch.full((1024, filler // 1024), 9, dtype=torch.uint8, device="cuda"),
                       "out_xy": torch.empty((corners, 2), device="cuda"),
                       "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")})
    ctx = lk.lk_context_create(0, 0)
    try:
        det = lk.lk_detector_create(ctx, len(frames), sum(f["img"].numel() for f in frames))
        lk.lk_detect_corners(det, frames, lk.gftt_params(1, 0, corners, border, quality))
        torch.cuda.synchronize()
        for size, f, xy in zip(SIZES, frames, want):
            got = f["out_xy"][:int(f["count"].item())].cpu().numpy()
            assert np.array_equal(got, xy), size
        if filler:
            assert int(frames[-1]["count"].item()) == 0
        lk.lk_detector_destroy(det)
    finally:
        lk.lk_context_destroy(ctx)
