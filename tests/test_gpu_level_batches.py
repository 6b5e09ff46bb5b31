"""The tracker's launch with a wavefront per pyramid level, in batches: several
frame pairs of different sizes, keypoint counts on both sides of its limits,
end points written over the start points, and a pool whose live counts lie
below its capacity.  Everywhere the same bits as a wavefront per keypoint."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SIZES = [(320, 240), (97, 83), (200, 150), (33, 40)]
FILL = 3200                      # points that move a launch past every limit


# (window, levels, binary16, keypoints in all): at the limit and one past it
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("win,levels,f16,n", [
    (21, 2, 0, 2048), (21, 3, 0, 1280), (21, 3, 0, 1281), (21, 4, 0, 1024), (9, 3, 0, 600),
    (21, 3, 1, 1706), (21, 3, 1, 1707), (15, 4, 1, 1280), (31, 3, 1, 768), (31, 4, 1, 640), (31, 4, 1, 641),
    (31, 2, 0, 768), (31, 3, 0, 512)])
def test_batches(win, levels, f16, n, in_place):
    import torch
    from paper_2607_01757_amd import lk

    print(win, levels, f16, n, in_place, flush=True)
    rng = np.random.default_rng(n + win)
    ctx = lk.lk_context_create(0, 0)
    try:
        pyrs, pts, counts = [], [], [n // 2, 0, n - n // 2 - 7, 7]
        for k, (w, h) in enumerate(SIZES):
            pr = synth.pair(20 + k, w, h, 8)
            pair = []
            for im in (pr.prev, pr.next):
                p, t = lk.lk_pyramid_create(ctx, w, h, levels, f16), torch.from_numpy(im).cuda()
                lk.lk_build_pyramid(ctx, p, t)
                pair.append((p, t))
            pyrs.append(pair)
            q = rng.uniform([-2, -2], [w + 1, h + 1], (counts[k], 2)).astype(np.float32)      # a few outside
            pts.append(q)
        fill = rng.uniform([0, 0], [SIZES[0][0] - 1, SIZES[0][1] - 1], (FILL, 2)).astype(np.float32)
        start = torch.from_numpy(np.concatenate(pts + [fill])).cuda()
        offs = np.concatenate([[0], np.cumsum(counts)]).astype(int)
        items = [(a[0][0], a[1][0], int(o), c) for a, o, c in zip(pyrs, offs, counts)]
        prm = lk.make_params(win, levels, 30, 0.01, 1e-6, 1.0)

        def track(pairs):
            out = [t.zero_() for t in lk.outputs(n + FILL, levels, with_iters=True)]
            src = start.clone()
            if in_place:
                out[0] = src
            lk.lk_track_batched(ctx, pairs, src, None, prm, *out)
            return [t[:n].cpu().numpy() for t in out]

        ref = track(items + [(pyrs[0][0][0], pyrs[0][1][0], n, FILL)])
        got = track(items)
        for name, a, b in zip(("points", "status", "residual", "iterations"), got, ref):
            assert a.tobytes() == b.tobytes(), name
        assert 0 < (ref[1] == 0).sum() < n
        for pair in pyrs:
            for p, _ in pair:
                lk.lk_pyramid_destroy(p)
    finally:
        lk.lk_context_destroy(ctx)


def test_live_counts():
    """One camera's pool (capacity 256, at most 60 tracks: a wavefront per
    level) against the same camera among 12 (a wavefront per keypoint)."""
    import torch
    from paper_2607_01757_amd import lk

    ctx = lk.lk_context_create(0, 0)
    try:
        got = []
        for n in (1, 12):
            cap, (w, h) = 256, (320, 240)
            state, scratch = lk.pool_state(n, cap), lk.pool_scratch(n, cap)
            pool = lk.lk_pool_create(ctx, n, cap, n * w * h, state, scratch)
            pyr = [[lk.lk_pyramid_create(ctx, w, h, 3, 0) for _ in range(2)] for _ in range(n)]
            keep, states = [], []
            prm, det = lk.make_params(21, 3, 30, 0.01, 1e-6, 1.0), lk.gftt_params(1, 20, 60, 8, 0.01)
            for t in range(4):
                frames = []
                for i in range(n):
                    pr = synth.pair(40 + i, w, h, 8)
                    im = torch.from_numpy(pr.next if t & 1 else pr.prev).cuda()
                    lk.lk_build_pyramid(ctx, pyr[i][t & 1], im)
                    keep.append(im)
                    frames.append((i, pyr[i][(t - 1) & 1] if t else None, pyr[i][t & 1], None))
                lk.lk_pool_step(pool, frames, prm, None, det)
                c = int(state["count"][0].item())
                assert 0 < c <= 60
                states.append((c, state["pts"][0, :c].cpu().numpy().tobytes(), state["ids"][0, :c].cpu().numpy().tobytes()))
            got.append(states)
            lk.lk_pool_destroy(pool)
            for a in pyr:
                for p in a:
                    lk.lk_pyramid_destroy(p)
        assert got[0] == got[1]
    finally:
        lk.lk_context_destroy(ctx)
