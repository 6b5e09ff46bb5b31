"""Detection on frames whose rows lie far apart (pitch * h of 2 GiB and more,
where 32-bit offsets wrap): the corners and the response map of the same frame
with compact rows, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

W, H = 208, 32768


@pytest.mark.parametrize("pitch", [65536, 131072, 163840])      # 2, 4 and 5 GiB
@pytest.mark.parametrize("radius,response", [(0, True), (1, False), (1, True), (2, True), (3, False)])
def test_far_rows(radius, response, pitch):
    import torch
    from paper_2607_01757_amd import lk

    print(radius, response, pitch, flush=True)
    rng = np.random.default_rng(radius)
    im = torch.from_numpy(rng.integers(0, 256, (H, W), dtype=np.uint8)).cuda()
    far = torch.empty((H, pitch), dtype=torch.uint8, device="cuda")[:, :W]
    far.copy_(im)
    ctx = lk.lk_context_create(0, 0)
    try:
        det = lk.lk_detector_create(ctx, 1, W * H)
        got = []
        for img in (im, far):
            f = {"img": img, "out_xy": torch.full((4096, 2), -1.0, device="cuda"),
                 "count": torch.full((1,), -1, dtype=torch.int32, device="cuda")}
            if response:
                f["response"] = torch.full((H, W), -1.0, dtype=torch.float64, device="cuda")
            lk.lk_detect_corners(det, [f], lk.gftt_params(radius, 0, 4096, 0, 0.0))
            torch.cuda.synchronize()
            got.append(f)
        a, b = got
        assert int(a["count"].item()) == 4096 or radius == 0    # (radius 0: every response is 0)
        if radius:
            assert bool((a["out_xy"][:, 1] > H // 2).any())     # corners past 2 GiB are among them
        assert int(a["count"].item()) == int(b["count"].item())
        assert torch.equal(a["out_xy"], b["out_xy"])
        if response:
            assert torch.equal(a["response"].view(torch.int64), b["response"].view(torch.int64))
        lk.lk_detector_destroy(det)
    finally:
        lk.lk_context_destroy(ctx)
