"""Selection on plateaus: thousands of equal responses, so that windows end in
the index digits of the rank key after many passes, at several candidates a
window's capacity (2048) and spacings, against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("min_dist,corners", [(0, 4096), (2, 4096), (8, 1000), (30, 200)])
@pytest.mark.parametrize("cell,w,h", [(8, 320, 240), (8, 752, 480), (5, 411, 333), (16, 640, 480)])
def test_plateaus(cell, w, h, min_dist, corners):
    import torch
    from paper_2607_01757_amd import lk

    print(cell, w, h, min_dist, corners, flush=True)
    y, x = np.mgrid[0:h, 0:w]
    checks = np.where(((x // cell) + (y // cell)) % 2, 255, 0).astype(np.uint8)
    mixed = checks.copy()                      # plateaus of many levels, row by row
    mixed[(y // cell) % 3 == 1] //= 2
    ims = [checks, mixed, np.where(x % 37 < 12, checks, 255 - checks // 3)]
    ctx = lk.lk_context_create(0, 0)
    try:
        det = lk.lk_detector_create(ctx, len(ims), len(ims) * w * h)
        frames = [{"img": torch.from_numpy(np.ascontiguousarray(im)).cuda(),
                   "out_xy": torch.full((corners, 2), -1.0, device="cuda"),
                   "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")} for im in ims]
        lk.lk_detect_corners(det, frames, lk.gftt_params(1, min_dist, corners, 0, 0.01))
        torch.cuda.synchronize()
        for im, f in zip(ims, frames):
            want = np.asarray(oracle.gftt(im, r=1, quality=0.01, min_dist=min_dist, max_corners=corners, border=0)).reshape(-1, 2)
            got = f["out_xy"][:int(f["count"].item())].cpu().numpy()
            assert np.array_equal(got, want)
        lk.lk_detector_destroy(det)
    finally:
        lk.lk_context_destroy(ctx)
