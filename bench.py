#!/usr/bin/env python3
"""Benchmark of the pyramidal LK hot path on one MI355X.

Default workload ("batched"): 64 independent camera streams, resolution
uniform over {640x480, 752x480, 960x600, 1280x720, 1920x1080}, U[150, 1500]
keypoints per frame, sub-pixel shifts up to 8 px with noise sigma 2;
21x21 window, 3 levels, 30 iterations, eps 0.01, float32 storage.  One step
is the steady state of all streams: the new frame of every stream gets its
pyramid (one launch per level for all frames) and every keypoint is tracked
from the resident previous pyramid in one launch.  The same frames are also
run through the plain per-frame path (one pyramid build and one tracker
launch per stream) for comparison.

Prints one JSON line on stdout; progress goes to stderr.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0          # MI355X HBM3E, GB/s
PEAK_FP32_TFLOPS = 157.3       # MI355X fp32 vector (packed); 78.6 without packed FP32
# algorithmic flops per window pixel: 29 per level for the template (three
# bilinear samples, the normal matrix), 13 per Gauss-Newton iteration (one
# bilinear sample, the mismatch and its two products)
FLOP_TEMPLATE, FLOP_ITER = 29, 13


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def percentile(xs, q):
    return float(np.percentile(np.asarray(xs), q)) if len(xs) else 0.0


def level_dims(w, h, levels):
    out = [(w, h)]
    for _ in range(1, levels):
        w, h = (w + 1) // 2, (h + 1) // 2
        out.append((w, h))
    return out


def footprint_bytes(pts, ends, w, h, levels, win, store_bytes, grad_bytes=0):
    """Unique bytes of the window footprints the tracker must read: template
    windows (win+3)^2 around p / 2^l in the previous pyramid (plus the
    gradient planes of levels >= 1, grad_bytes per pixel, when they are
    stored) and target windows (win+1)^2 covering start and end in the next
    one."""
    hw = (win - 1) // 2
    total = 0
    for l, (lw, lh) in enumerate(level_dims(w, h, levels)):
        for pts_l, ext in ((pts / 2 ** l, hw + 2), (None, hw + 1)):
            s = (1 if l == 0 else store_bytes) + (grad_bytes if pts_l is not None and l > 0 else 0)
            diff = np.zeros((lh + 1, lw + 1), np.int32)
            if pts_l is not None:
                x0 = np.floor(pts_l[:, 0]) - ext + 1
                x1 = np.floor(pts_l[:, 0]) + ext + 1
                y0 = np.floor(pts_l[:, 1]) - ext + 1
                y1 = np.floor(pts_l[:, 1]) + ext + 1
            else:
                a, b = pts / 2 ** l, ends / 2 ** l
                lo, hi = np.minimum(a, b), np.maximum(a, b)
                x0 = np.floor(lo[:, 0]) - ext
                x1 = np.floor(hi[:, 0]) + ext + 2
                y0 = np.floor(lo[:, 1]) - ext
                y1 = np.floor(hi[:, 1]) + ext + 2
            x0 = np.clip(x0, 0, lw).astype(int); x1 = np.clip(x1, 0, lw).astype(int)
            y0 = np.clip(y0, 0, lh).astype(int); y1 = np.clip(y1, 0, lh).astype(int)
            np.add.at(diff, (y0, x0), 1); np.add.at(diff, (y0, x1), -1)
            np.add.at(diff, (y1, x0), -1); np.add.at(diff, (y1, x1), 1)
            cover = np.cumsum(np.cumsum(diff, 0), 1)[:lh, :lw] > 0
            total += int(cover.sum()) * s
    return total


def flops_from_iters(iters, win, fb):
    """Algorithmic flops of the tracker from per-point iteration counts
    (N x 2 x L: forward / backward)."""
    nw = win * win
    it = iters.astype(np.int64)
    L = it.shape[2]
    passes = 1 + (1 if fb else 0)
    per = nw * FLOP_TEMPLATE * L * passes
    return float(len(it) * per + nw * FLOP_ITER * it.sum())


# ---------------------------------------------------------------- workloads

def make_streams(n_streams, seed):
    import synth
    t0 = time.time()
    streams = synth.batch_streams(seed, n_streams=n_streams)
    log("generated %d streams in %.1fs (%d keypoints)" % (n_streams, time.time() - t0,
                                                        sum(len(s.pts) for s in streams)))
    return streams


class BatchedWorkload:
    def __init__(self, lk, ctx, streams, win=21, levels=3, storage=0, fb=0.0):
        import torch
        self.lk, self.ctx, self.streams = lk, ctx, streams
        self.win, self.levels, self.storage, self.fb = win, levels, storage, fb
        self.prev_img = [torch.from_numpy(s.prev).cuda() for s in streams]
        self.next_img = [torch.from_numpy(s.next).cuda() for s in streams]
        self.prev_pyr = [lk.lk_pyramid_create(ctx, s.width, s.height, levels, storage) for s in streams]
        self.next_pyr = [lk.lk_pyramid_create(ctx, s.width, s.height, levels, storage) for s in streams]
        lk.lk_build_pyramids(ctx, self.prev_pyr, self.prev_img)
        counts = [len(s.pts) for s in streams]
        self.offsets = np.concatenate([[0], np.cumsum(counts)[:-1]]).astype(np.int64)
        self.n = int(sum(counts))
        self.pts = torch.from_numpy(np.concatenate([s.pts for s in streams])).cuda()
        self.pairs = [(a, b, int(o), c) for a, b, o, c in zip(self.prev_pyr, self.next_pyr, self.offsets, counts)]
        self.params = lk.make_params(win, levels, 30, 0.01, 1e-6, fb)
        self.out, self.st, self.res, self.it = lk.outputs(self.n, levels, with_iters=True)
        torch.cuda.synchronize()

    def build(self):
        self.lk.lk_build_pyramids(self.ctx, self.next_pyr, self.next_img)

    def time_build(self, reps, warmup):
        """Device time of the new-frame pyramids of every stream: a prepared,
        graph-captured batch with no pairs, replayed back to back."""
        lk = self.lk
        b = lk.lk_batch_create(self.ctx, self.next_pyr, self.next_img, [], self.pts, None, self.params, self.out,
                               self.st, self.res, None, config=lk.lk_exec_config(0, 0, 1, 0))
        t = time_block(lambda: lk.lk_batch_run(b), reps, warmup)
        lk.lk_batch_destroy(b)
        return t

    def track(self, iters=False):
        self.lk.lk_track_batched(self.ctx, self.pairs, self.pts, None, self.params, self.out, self.st,
                                 self.res, self.it if iters else None)

    def step(self):
        self.build()
        self.track()

    def plain_frame(self, i):
        lk, s = self.lk, self.streams[i]
        lk.lk_build_pyramid(self.ctx, self.next_pyr[i], self.next_img[i])
        o, c = int(self.offsets[i]), len(s.pts)
        lk.lk_track(self.ctx, self.prev_pyr[i], self.next_pyr[i], self.pts[o:o + c], None, c, self.params,
                    self.out[o:o + c], self.st[o:o + c], self.res[o:o + c], None)

    def close(self):
        for p in self.prev_pyr + self.next_pyr:
            self.lk.lk_pyramid_destroy(p)


def settle(fn, seconds=0.15):
    """Runs fn back to back for about `seconds` of device time, untimed: the
    GPU's clock rises over the first tens of milliseconds of sustained work
    (the tracker's kernel time falls from about 180 to 157 us over 25 ms), so
    timed regions start from the steady clock a busy device runs at."""
    import torch
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    while time.perf_counter() - t0 < seconds:
        for _ in range(8):
            fn()
        torch.cuda.synchronize()


def prepared_step(lk, ctx, build_pyrs, build_imgs, pairs, pts, params, out, st, res):
    """A graph-captured prepared step with the execution shape of the
    committed table of tuned shapes (lk_exec_table.txt), or of the autotuner
    when the table has no row for this batch."""
    cfg, found = lk.lk_exec_table_lookup(ctx, pairs, params)
    step = lk.lk_batch_create(ctx, build_pyrs, build_imgs, pairs, pts, None, params, out, st, res, None,
                              config=None if found else lk.lk_exec_config(0, 0, 1, 0, 0, 0))
    if found:
        best, source = lk.lk_batch_config(step), "table"
    else:
        best, _ = lk.lk_batch_tune(step, reps=3)
        source = "autotuner"
    log("execution shape (%s): persistent=%d blocks_per_cu=%d chunk=%d waves_per_group=%d" % (
        source, best.persistent, best.blocks_per_cu, best.chunk, best.waves_per_group))
    return step, best, source


def time_steps(fn, steps, warmup):
    import torch
    settle(fn)
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    t0 = time.perf_counter()
    for a, b in evs:
        a.record()
        fn()
        b.record()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    per = [a.elapsed_time(b) for a, b in evs]
    return wall, per


def time_block(fn, reps, warmup):
    """Mean duration of one call when `reps` calls run back to back, from two
    HIP events on the launch stream around the whole run."""
    import torch
    settle(fn)
    for _ in range(warmup):
        fn()
    torch.cuda.synchronize()
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    a.record()
    for _ in range(reps):
        fn()
    b.record()
    torch.cuda.synchronize()
    return a.elapsed_time(b) / reps * 1e-3


def profiled_traffic(kernel, summary="profiles/hbm_counters_batched64.txt",
                     source="paper_2607_01757_amd/csrc/lk_kernels.hip"):
    """HBM bytes per launch of `kernel` from the committed rocprofv3 counter
    summary (FETCH_SIZE + WRITE_SIZE, copy-calibrated), or None when the
    kernel source has changed since the counters were taken."""
    import hashlib
    root = os.path.dirname(os.path.abspath(__file__))
    try:
        lines = open(os.path.join(root, summary)).read().splitlines()
        now = hashlib.sha256(open(os.path.join(root, source), "rb").read()).hexdigest()
    except OSError:
        return None
    recorded = [l.split()[2] for l in lines if l.startswith("source sha256") and l.split()[3] == source]
    if recorded != [now]:
        return None
    for l in lines:
        f = l.split()
        if len(f) == 3 and f[0] == "traffic" and f[1] == kernel:
            return int(f[2])
    return None


def detect_traffic():
    """HBM bytes of one 64-frame detection step: the sum over its kernels of
    the copy-calibrated counter summary, or None when a kernel is missing
    from it or the detector source has changed since (the reset kernel, a
    fill of 2 KiB per frame, is left out)."""
    parts = [profiled_traffic(k, summary="profiles/hbm_counters_detect64.txt",
                              source="paper_2607_01757_amd/csrc/lk_gftt.hip")
             for k in ("k_gftt_peaks_pair", "k_gftt_compact", "k_gftt_bucket", "k_gftt_select")]
    return None if any(v is None for v in parts) else sum(parts)


def cpu_baseline(streams, n_sample, win, levels, fb, n_sample_1t=16):
    """The FP64 oracle timed on the host: on every core over n_sample streams,
    and on one thread over the first n_sample_1t of them."""
    import oracle
    threads = os.cpu_count() or 1

    def timed(sample, nthreads):
        npts = sum(len(s.pts) for s in sample)
        t0 = time.perf_counter()
        for s in sample:
            oracle.track(s.prev, s.next, s.pts, win=win, levels=levels, min_eig=1e-6, fb_thresh=fb,
                         nthreads=nthreads)
        return npts, time.perf_counter() - t0

    npts, dt = timed(streams[:n_sample], threads)
    n1, dt1 = timed(streams[:n_sample_1t], 1)
    return {"value": npts / dt, "unit": "keypoints/s", "cores": threads, "kind": "oracle",
            "sample": "%d of %d streams, all %d of their keypoints; the oracle builds both pyramids of "
                      "each pair (FP64) and tracks on %d threads; %.1f s wall" % (n_sample, len(streams), npts,
                                                                                  threads, dt),
            "one_thread": {"value": n1 / dt1, "unit": "keypoints/s", "cores": 1,
                           "sample": "the first %d streams, %d keypoints, %.1f s wall" % (n_sample_1t, n1, dt1)}}


def copy_bandwidth(nbytes=1 << 30, reps=20):
    """Attainable HBM bandwidth: a device-to-device copy of nbytes, timed
    with HIP events over reps back-to-back copies (read + write bytes)."""
    import torch
    a = torch.empty(nbytes, dtype=torch.uint8, device="cuda").fill_(1)
    b = torch.empty_like(a)
    t = time_block(lambda: b.copy_(a), reps, 3)
    del a, b
    torch.cuda.empty_cache()
    return 2.0 * nbytes / t / 1e9


def run_batched(args):
    import torch
    from paper_2607_01757_amd import lk

    streams = make_streams(args.streams, args.seed)
    ctx = lk.lk_context_create(0, 0)
    f16 = args.storage == "f16"
    wl = BatchedWorkload(lk, ctx, streams, storage=lk.LK_STORAGE_F16 if f16 else lk.LK_STORAGE_F32)
    log("resident: %.1f MB of pyramids, %d keypoints" % (lk.lk_context_bytes_in_use(ctx) / 1e6, wl.n))
    # one untimed step with iteration counts (deterministic: same counts when timed)
    wl.step()
    wl.track(iters=True)
    torch.cuda.synchronize()
    iters = wl.it.cpu().numpy()
    status = wl.st.cpu().numpy()
    ends = wl.out.cpu().numpy()
    f_alg = flops_from_iters(iters, wl.win, False)

    # the step as one prepared batch: new-frame pyramids + all pairs, recorded
    # into a HIP graph, execution shape from the committed table of tuned
    # shapes (the autotuner runs here only when the table has no row for it)
    step, best, shape_source = prepared_step(lk, ctx, wl.next_pyr, wl.next_img, wl.pairs, wl.pts, wl.params,
                                             wl.out, wl.st, wl.res)
    # the tracker alone, same shape, for the roofline of the dominant kernel:
    # direct launches back to back (a graph replay per launch would add its
    # own gap to every kernel)
    trk = lk.lk_batch_create(ctx, [], [], wl.pairs, wl.pts, None, wl.params, wl.out, wl.st, wl.res, None,
                             config=lk.lk_exec_config(best.persistent, best.blocks_per_cu, 0, best.chunk,
                                                      best.waves_per_group, 0))
    t_trk = time_block(lambda: lk.lk_batch_run(trk), max(args.steps, 10), args.warmup)
    t_pyr = wl.time_build(max(args.steps, 10), args.warmup)
    wall, per = time_steps(lambda: lk.lk_batch_run(step), args.steps, args.warmup)
    kps = wl.n * args.steps / wall
    log("batched (graph): %.3f ms/step  %.3g kp/s  tracker %.3f ms  pyramids %.3f ms" %
        (wall / args.steps * 1e3, kps, t_trk * 1e3, t_pyr * 1e3))
    # the same step through the unprepared batched calls (tables shipped per call)
    uw, _ = time_steps(wl.step, args.steps, args.warmup)
    unprepared = {"value": wl.n * args.steps / uw, "unit": "keypoints/s", "ms_per_step": uw / args.steps * 1e3}

    # plain per-frame launches over the same frames
    plain = None
    if not args.no_plain:
        def plain_step():
            for i in range(len(streams)):
                wl.plain_frame(i)
        k = max(2, args.steps // 4)
        pw, pper = time_steps(plain_step, k, max(1, args.warmup // 2))
        # per-frame latency of the plain path: each frame alone, events around it
        lat = []
        for i in range(len(streams)):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(); wl.plain_frame(i); b.record()
            torch.cuda.synchronize()
            lat.append(a.elapsed_time(b))
        # frames of one step arriving together: completion time of each
        # frame when the plain path runs them one after another
        evs = [torch.cuda.Event(enable_timing=True) for _ in range(len(streams) + 1)]
        evs[0].record()
        for i in range(len(streams)):
            wl.plain_frame(i)
            evs[i + 1].record()
        torch.cuda.synchronize()
        done = [evs[0].elapsed_time(e) for e in evs[1:]]
        plain = {"value": wl.n * k / pw, "unit": "keypoints/s", "ms_per_step": pw / k * 1e3,
                 "p50_frame_ms": percentile(lat, 50), "p99_frame_ms": percentile(lat, 99),
                 "step_completion_p50_ms": percentile(done, 50), "step_completion_p99_ms": percentile(done, 99)}
        log("plain: %.3f ms/step  %.3g kp/s" % (plain["ms_per_step"], plain["value"]))

    # algorithmic bytes of one step (whole path)
    b_frames = sum(s.width * s.height for s in streams)
    esz = 2 if f16 else 4
    b_levels = sum(esz * sum(w * h for (w, h) in level_dims(s.width, s.height, 3)[1:]) for s in streams)
    if f16:   # binary16 gradient planes of levels >= 1 (4 B per pixel)
        b_levels += sum(4 * sum(w * h for (w, h) in level_dims(s.width, s.height, 3)[1:]) for s in streams)
    b_windows = 0
    off = 0
    for s in streams:
        c = len(s.pts)
        b_windows += footprint_bytes(s.pts.astype(np.float64), ends[off:off + c].astype(np.float64),
                                     s.width, s.height, 3, 21, esz, 4 if f16 else 0)
        off += c
    b_io = wl.n * (8 + 8 + 1 + 4)
    b_alg = b_frames + b_levels + b_windows + b_io
    step_s = wall / args.steps
    copy_gbs = copy_bandwidth()
    log("device copy: %.0f GB/s (read + write)" % copy_gbs)

    result = {
        "metric": "tracked keypoints/sec (batched, 64 streams) + p50/p99 frame latency",
        "value": kps, "unit": "keypoints/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": step_s * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16" if f16 else "f32", "data": "synthetic",
        "config": {"workload": "batched: 64 streams, resolutions {640x480..1920x1080}, U[150,1500] keypoints, "
                               "21x21 window, 3 levels, 30 iterations, eps 0.01, %s storage; one step = " % (
                                   "binary16" if f16 else "float32") +
                               "new-frame pyramids + all pairs in one graph-captured prepared batch",
                   "streams": len(streams), "keypoints_per_step": wl.n, "seed": args.seed,
                   "exec": {"persistent": best.persistent, "blocks_per_cu": best.blocks_per_cu,
                            "chunk": best.chunk, "waves_per_group": best.waves_per_group, "use_graph": 1,
                            "source": shape_source}},
        "p50_frame_ms": percentile(per, 50), "p99_frame_ms": percentile(per, 99),
        "tracked_fraction": float(np.mean(status == 0)),
        "roofline": {"bound": "alu", "kernel": "k_track_%s" % ("persist" if best.persistent else "batched"),
                     "achieved": f_alg / t_trk / 1e12, "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s",
                     "frac": f_alg / t_trk / 1e12 / PEAK_FP32_TFLOPS,
                     "traffic": profiled_traffic("k_track_batched", summary="profiles/hbm_counters_batched64%s.txt"
                                                 % ("_f16" if f16 else "")),
                     "flops_per_launch": f_alg, "kernel_ms": t_trk * 1e3},
        "path_hbm": {"algorithmic_bytes": b_alg, "achieved_GBs": b_alg / step_s / 1e9,
                     "frac": b_alg / step_s / 1e9 / PEAK_HBM_GBS,
                     "copy_GBs": copy_gbs, "frac_of_copy": b_alg / step_s / 1e9 / copy_gbs},
        "pyramid_ms": t_pyr * 1e3,
        "unprepared_batched": unprepared,
        "plain": plain,
    }
    if not args.no_cpu_baseline:
        log("timing the CPU oracle on a sample ...")
        result["cpu_baseline"] = cpu_baseline(streams, args.cpu_streams, 21, 3, 0.0)
    lk.lk_batch_destroy(step)
    lk.lk_batch_destroy(trk)
    wl.close()
    lk.lk_context_destroy(ctx)
    return result


_SEQ = None


def _render_init(seed, nf, gain_mode):
    global _SEQ
    import synth
    _SEQ = synth.StereoSequence(seed, n_frames=nf, gain_mode=gain_mode)


def _render_frame(t):
    return _SEQ.frame(t, 0), _SEQ.frame(t, 1)


def render_stereo(seed, nf, gain_mode):
    """Both cameras of frames 0 .. nf-1, rendered by a pool of host processes
    (forked before this process touches the GPU)."""
    import multiprocessing as mp
    workers = max(1, min(16, os.cpu_count() or 1))
    if workers == 1 or nf < 32:
        _render_init(seed, nf, gain_mode)
        frames = [_render_frame(t) for t in range(nf)]
    else:
        with mp.get_context("fork").Pool(workers, initializer=_render_init, initargs=(seed, nf, gain_mode)) as pool:
            frames = pool.map(_render_frame, range(nf), chunksize=8)
    return [f[0] for f in frames], [f[1] for f in frames]


def _pass_error(records, frames_a, frames_b, win, levels, label):
    """Every recorded tracker call of one pass against the FP64 oracle
    (unrounded pyramids): end-point error over points both track, and status
    agreement over all points."""
    import oracle
    errs, agree, total, both = [], 0, 0, 0
    t0 = time.time()
    for k, (t, p0, g_pts, g_st) in enumerate(records):
        r = oracle.track(frames_a(t), frames_b(t), p0, win=win, levels=levels, fb_thresh=1.0, min_eig=1e-6,
                         nthreads=os.cpu_count() or 1)
        ok = (g_st == 0) & (r.status == 0)
        errs.append(np.abs(g_pts[ok] - r.pts[ok]).max(axis=1))
        agree += int(np.sum(g_st == r.status))
        total += len(g_st)
        both += int(ok.sum())
        if (k + 1) % 200 == 0:
            log("  %s pass: %d / %d frames against the oracle (%.0f s)" % (label, k + 1, len(records),
                                                                          time.time() - t0))
    e = np.concatenate(errs) if errs else np.zeros(0)
    return {"frames": len(records), "points": total, "tracked_by_both": both,
            "max_px": float(e.max()) if e.size else 0.0, "p99_px": float(np.percentile(e, 99)) if e.size else 0.0,
            "over_1e-3_px": int(np.sum(e > 1e-3)), "over_1e-2_px": int(np.sum(e > 1e-2)),
            "status_agreement": agree / total if total else 1.0, "status_differs": total - agree}


def run_stereo(args, f16):
    """Stereo sequence: per frame, pyramids of the left and right frames,
    temporal tracking (left t-1 -> t) and stereo tracking (left -> right),
    both with a 1 px forward-backward check; 200 keypoints per frame
    (survivors carried, topped up with new points).  Plain per-frame
    launches, and the same two pairs as one batch of two.  Every tracker
    call of the timed run is then compared with the FP64 oracle (both
    passes, every frame)."""
    import torch
    import synth
    from paper_2607_01757_amd import lk

    win, levels = (31, 4) if f16 else (21, 4)
    storage = lk.LK_STORAGE_F16 if f16 else lk.LK_STORAGE_F32
    nf = args.frames
    seq = synth.StereoSequence(args.seed, n_frames=max(nf, 2), gain_mode=args.gain_mode)
    t_r = time.time()
    left, right = render_stereo(args.seed, max(nf, 2), args.gain_mode)
    log("rendered %d stereo frames in %.1fs" % (nf, time.time() - t_r))
    ctx = lk.lk_context_create(0, 0)
    W, H = seq.width, seq.height
    dl = [torch.from_numpy(f).cuda() for f in left]
    dr = [torch.from_numpy(f).cuda() for f in right]
    pl = [lk.lk_pyramid_create(ctx, W, H, levels, storage) for _ in range(2)]
    pr = lk.lk_pyramid_create(ctx, W, H, levels, storage)
    prm = lk.make_params(win, levels, 30, 0.01, 1e-6, 1.0)
    N = 200
    outs = [lk.outputs(N, levels) for _ in range(2)]
    d_pts = torch.empty((2 * N, 2), dtype=torch.float32, device="cuda")

    def run(mode, record):
        rng = np.random.default_rng(args.seed)
        pts = synth.uniform_points(rng, N, W, H)
        lk.lk_build_pyramid(ctx, pl[0], dl[0])
        torch.cuda.synchronize()
        lat, kp, temporal, stereo = [], 0, [], []
        t0 = time.perf_counter()
        for t in range(1, nf):
            a, b = pl[(t - 1) & 1], pl[t & 1]
            ts = time.perf_counter()
            p_in = pts
            d_pts[:N].copy_(torch.from_numpy(pts))
            if mode == "plain":
                lk.lk_build_pyramid(ctx, b, dl[t])
                lk.lk_build_pyramid(ctx, pr, dr[t])
            else:
                lk.lk_build_pyramids(ctx, [b, pr], [dl[t], dr[t]])
            lk.lk_track(ctx, a, b, d_pts[:N], None, N, prm, *outs[0][:3], None)
            st = outs[0][1].cpu().numpy()
            q = outs[0][0].cpu().numpy()
            if record:
                temporal.append((t, p_in.copy(), q.astype(np.float64), st.copy()))
            keep = q[st == 0]
            keep = keep[(keep[:, 0] >= 16) & (keep[:, 0] <= W - 17) & (keep[:, 1] >= 16) & (keep[:, 1] <= H - 17)]
            new = synth.uniform_points(rng, N - len(keep), W, H)
            pts = np.concatenate([keep, new]).astype(np.float32)[:N]
            d_pts[N:].copy_(torch.from_numpy(pts))
            lk.lk_track(ctx, b, pr, d_pts[N:], None, N, prm, *outs[1][:3], None)
            st2 = outs[1][1].cpu().numpy()
            if record:
                stereo.append((t, pts.copy(), outs[1][0].cpu().numpy().astype(np.float64), st2.copy()))
            lat.append((time.perf_counter() - ts) * 1e3)
            kp += 2 * N
        wall = time.perf_counter() - t0
        return kp / wall, lat, temporal, stereo

    run("plain", False)                                   # warm-up
    kps, lat, temporal, stereo = run("plain", True)
    kps_b, lat_b, _, _ = run("batch2", False)
    log("stereo %s (%s gains): plain %.3g kp/s p50 %.3f ms p99 %.3f ms; left+right pyramids in one launch %.3g kp/s "
        "p99 %.3f ms" % ("f16" if f16 else "f32", args.gain_mode, kps, percentile(lat, 50), percentile(lat, 99),
                         kps_b, percentile(lat_b, 99)))
    result = {
        "metric": "tracked keypoints/sec + p50/p99 frame latency (stereo sequence, plain per-frame)",
        "value": kps, "unit": "keypoints/s", "n_gpus": 1, "steps": nf - 1, "warmup": nf - 1,
        "ms_per_step": float(np.mean(lat)), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16" if f16 else "f32", "data": "synthetic",
        "config": {"workload": "stereo sequence 752x480, %d frames, %s gains, 200 keypoints, temporal + "
                               "left-to-right with FB 1 px, %dx%d, 4 levels, %s storage" % (
                                   nf, args.gain_mode, win, win, "binary16" if f16 else "float32")},
        "p50_frame_ms": percentile(lat, 50), "p99_frame_ms": percentile(lat, 99),
        "batch2": {"value": kps_b, "p50_frame_ms": percentile(lat_b, 50), "p99_frame_ms": percentile(lat_b, 99)},
    }
    for p_ in pl + [pr]:
        lk.lk_pyramid_destroy(p_)
    lk.lk_context_destroy(ctx)
    if args.precision_frames != 0:
        nrec = len(temporal) if args.precision_frames < 0 else min(args.precision_frames, len(temporal))
        log("comparing %d frames of both passes with the FP64 oracle (unrounded pyramids) ..." % nrec)
        err = {
            "temporal": _pass_error(temporal[:nrec], lambda t: left[t - 1], lambda t: left[t], win, levels,
                                    "temporal"),
            "stereo": _pass_error(stereo[:nrec], lambda t: left[t], lambda t: right[t], win, levels, "stereo"),
        }
        result["error_vs_fp64_oracle_px"] = err
        for k, v in err.items():
            log("%s storage, %s pass vs FP64 oracle: max %.3g px p99 %.3g px over %d points tracked by both; "
                "status agrees on %.4f of %d" % ("binary16" if f16 else "float32", k, v["max_px"], v["p99_px"],
                                                   v["tracked_by_both"], v["status_agreement"], v["points"]))
    return result


def _serve_trace(args, literal):
    import synth
    res = ((752, 480),) if literal else synth.RESOLUTIONS
    return synth.ServingTrace(args.seed, n_streams=args.serve_streams,
                              duration_s=args.serve_warmup + args.serve_seconds, resolutions=res)


def serve_run(lk, ctx, trace, pool, pts, args, mode, rate_mult=1.0):
    """Drives one server with the trace's streams from args.serve_threads
    submitter threads (streams dealt round-robin; each thread also polls its
    own tickets).  mode "poisson": every frame is submitted at its scheduled
    arrival time (the trace compressed by rate_mult); latency = completion
    minus the scheduled arrival (both CLOCK_MONOTONIC), so submitter lag and
    busy retries count.  mode "closed": every stream keeps queue_depth frames
    outstanding for the whole run, which saturates the server; latency =
    completion minus the submit call's entry.  Returns the served results."""
    import ctypes as C
    import threading

    warm, dur = args.serve_warmup, args.serve_seconds
    prm16 = lk.make_params(31, 4, 30, 0.01, 1e-6, 1.0)
    qd = 4
    cfg = lk.server_config(max_streams=len(trace.streams), max_points=1500, levels=4, storage=lk.LK_STORAGE_F16,
                           params=prm16, max_batch=len(trace.streams), inflight=args.serve_inflight,
                           queue_depth=qd, hbm_budget_bytes=64 << 30)
    srv = lk.lk_server_create(ctx, cfg)
    ids = [lk.lk_server_open_stream(srv, sp.width, sp.height) for sp in trace.streams]
    resident = lk.lk_server_get_stats(srv).resident_bytes
    nthr = max(1, min(args.serve_threads, len(trace.streams)))
    mine = [[sp.stream for sp in trace.streams if sp.stream % nthr == t] for t in range(nthr)]
    events = [[e for e in trace.events if e[1] % nthr == t] for t in range(nthr)]
    results = [[] for _ in range(nthr)]        # (arrival_ns or submit_ns, done_ns, n, stream)
    busy = [0] * nthr
    t0_ns = time.monotonic_ns() + 50_000_000
    end_ns = t0_ns + int((warm + dur) * 1e9)

    def poll_some(tid, outstanding, block):
        n = C.c_int32()
        tm = lk.lk_timing()
        out = np.zeros((1500, 2), np.float32)
        st = np.zeros(1500, np.uint8)
        rs = np.zeros(1500, np.float32)
        while True:
            left = []
            for (t, ref_ns, sid) in outstanding:
                rc = lk.lib.lk_server_poll(srv, t, out.ctypes.data, st.ctypes.data, rs.ctypes.data, C.byref(n),
                                           C.byref(tm))
                if rc == lk.LK_ERR_NOT_READY:
                    left.append((t, ref_ns, sid))
                elif rc == lk.LK_SUCCESS:
                    results[tid].append((ref_ns if ref_ns else tm.submit_ns, tm.done_ns, n.value, sid))
                else:
                    raise RuntimeError("served frame failed: %d" % rc)
            outstanding[:] = left
            if not block or not outstanding:
                return
            time.sleep(0.0001)

    def submit(tid, sid, k):
        sp = trace.streams[sid]
        f = pool.frame(sp.width, sp.height, sid, k)
        while True:
            try:
                return lk.lk_server_submit(srv, ids[sid], f, pts[sid])
            except lk.LKError as e:
                if e.code != lk.LK_ERR_BUSY:
                    raise
                busy[tid] += 1
                time.sleep(0.0001)

    def poisson_worker(tid):
        outstanding = []
        for (ts, sid, k) in events[tid]:
            arrival = t0_ns + int(ts / rate_mult * 1e9)
            while time.monotonic_ns() < arrival:
                poll_some(tid, outstanding, False)
                time.sleep(0.00005)
            outstanding.append((submit(tid, sid, k), arrival, sid))
            if len(outstanding) > 8:
                poll_some(tid, outstanding, False)
        poll_some(tid, outstanding, True)

    def closed_worker(tid):
        outstanding = []
        nxt = {sid: 0 for sid in mine[tid]}
        while time.monotonic_ns() < t0_ns:
            time.sleep(0.0001)
        while time.monotonic_ns() < end_ns:
            count = {}
            for (_, _, sid) in outstanding:
                count[sid] = count.get(sid, 0) + 1
            for sid in mine[tid]:
                if count.get(sid, 0) < qd - 1:
                    outstanding.append((submit(tid, sid, nxt[sid]), 0, sid))
                    nxt[sid] += 1
            poll_some(tid, outstanding, False)
        poll_some(tid, outstanding, True)

    fn = poisson_worker if mode == "poisson" else closed_worker
    th = [threading.Thread(target=fn, args=(t,)) for t in range(nthr)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    stats = lk.lk_server_get_stats(srv)
    lk.lk_server_destroy(srv)
    done = [d for r in results for d in r]
    meas = [d for d in done if d[0] - t0_ns >= warm * 1e9 and d[2] > 0]
    lat = [(d[1] - d[0]) / 1e6 for d in meas]
    span = (max(d[1] for d in meas) - min(d[0] for d in meas)) / 1e9
    kp = sum(d[2] for d in meas)
    return {"value": kp / span, "unit": "keypoints/s", "frames_per_s": len(meas) / span,
            "p50_frame_ms": percentile(lat, 50), "p99_frame_ms": percentile(lat, 99),
            "max_frame_ms": float(max(lat)), "frames": len(meas), "batches": int(stats.batches),
            "frames_per_batch": stats.frames / max(1, stats.batches), "submit_busy_retries": int(sum(busy)),
            "submitter_threads": nthr, "resident_GB": resident / 1e9,
            "latency_from": "scheduled arrival" if mode == "poisson" else "submit call",
            "mode": mode if mode == "closed" else "poisson x%g" % rate_mult,
            "dtype": "f16 storage, f32 arithmetic"}


def run_serve(args):
    """256 camera streams with Poisson arrivals (U[20,30] Hz), resolution per
    stream from the batched set (or all 752x480 with --serve-res literal),
    U[150,1500] keypoints per frame, binary16 storage, 31x31, 4 levels,
    forward-backward 1 px: the offered trace, then a saturating closed-loop
    run (served capacity), then the same arrival trace through plain
    per-frame float32 launches."""
    import torch
    import synth
    from paper_2607_01757_amd import lk

    literal = args.serve_res == "literal"
    trace = _serve_trace(args, literal)
    res_set = ((752, 480),) if literal else synth.RESOLUTIONS
    pool = synth.FramePool(args.seed, resolutions=res_set)
    rng = np.random.default_rng(args.seed)
    pts = [synth.uniform_points(rng, sp.n_kp, sp.width, sp.height) for sp in trace.streams]
    warm, dur = args.serve_warmup, args.serve_seconds
    log("serving trace: %d streams, %d frames over %.0f s (%s resolutions)"
        % (len(trace.streams), len(trace.events), warm + dur, "752x480" if literal else "mixed"))
    ctx = lk.lk_context_create(0, 0)
    served = serve_run(lk, ctx, trace, pool, pts, args, "poisson", args.serve_rate_mult)
    log("served (offered load x%g): %.3g kp/s p50 %.2f ms p99 %.2f ms, %.1f frames/launch, %d busy retries"
        % (args.serve_rate_mult, served["value"], served["p50_frame_ms"], served["p99_frame_ms"],
           served["frames_per_batch"], served["submit_busy_retries"]))
    capacity = serve_run(lk, ctx, trace, pool, pts, args, "closed")
    log("served capacity (closed loop): %.3g kp/s (%.0f frames/s) p50 %.2f ms p99 %.2f ms, %.1f frames/launch"
        % (capacity["value"], capacity["frames_per_s"], capacity["p50_frame_ms"], capacity["p99_frame_ms"],
           capacity["frames_per_batch"]))

    # plain per-frame float32 launches driven by the same trace, one frame at a time
    prm32 = lk.make_params(31, 4, 30, 0.01, 1e-6, 1.0)
    pyr = {}
    dev_frames = {}
    pinned = {}
    d_pts = {}
    outs = lk.outputs(1500, 4)
    for sp in trace.streams:
        pyr[sp.stream] = [lk.lk_pyramid_create(ctx, sp.width, sp.height, 4, lk.LK_STORAGE_F32) for _ in range(2)]
        dev_frames[sp.stream] = [torch.empty((sp.height, sp.width), dtype=torch.uint8, device="cuda") for _ in range(2)]
        d_pts[sp.stream] = torch.from_numpy(pts[sp.stream]).cuda()
    for (w, h) in res_set:
        pinned[(w, h)] = torch.empty((h, w), dtype=torch.uint8).pin_memory()
    seen = {}
    lat2, kp2, t_first, t_last = [], 0, None, None
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for (ts, sid, k) in trace.events:
        now = time.perf_counter() - t0
        if now < ts:
            time.sleep(ts - now)
        sp = trace.streams[sid]
        cur = seen.get(sid, 0)
        hbuf = pinned[(sp.width, sp.height)]
        hbuf.numpy()[:] = pool.frame(sp.width, sp.height, sid, k)
        dev_frames[sid][cur & 1].copy_(hbuf, non_blocking=True)
        lk.lk_build_pyramid(ctx, pyr[sid][cur & 1], dev_frames[sid][cur & 1])
        if cur > 0:
            n = sp.n_kp
            lk.lk_track(ctx, pyr[sid][(cur - 1) & 1], pyr[sid][cur & 1], d_pts[sid], None, n, prm32,
                        outs[0], outs[1], outs[2], None)
            res = outs[0][:n].cpu()
            _ = res.numpy()
        torch.cuda.synchronize()
        tdone = time.perf_counter() - t0
        seen[sid] = cur + 1
        if ts >= warm and cur > 0:
            lat2.append((tdone - ts) * 1e3)
            kp2 += sp.n_kp
            t_first = ts if t_first is None else t_first
            t_last = tdone
    plain = {"value": kp2 / (t_last - t_first), "unit": "keypoints/s", "p50_frame_ms": percentile(lat2, 50),
             "p99_frame_ms": percentile(lat2, 99), "max_frame_ms": float(max(lat2)), "frames": len(lat2),
             "latency_from": "scheduled arrival", "dtype": "f32"}
    log("plain per-frame: %.3g kp/s p50 %.2f ms p99 %.2f ms" % (plain["value"], plain["p50_frame_ms"],
                                                                 plain["p99_frame_ms"]))
    for v in pyr.values():
        for p_ in v:
            lk.lk_pyramid_destroy(p_)
    lk.lk_context_destroy(ctx)
    span_ms = 1e3 * served["frames"] / max(served["frames_per_s"], 1e-9)
    return {
        "metric": "tracked keypoints/sec + p50/p99 frame latency (served, %d Poisson streams)" % len(trace.streams),
        "value": served["value"], "unit": "keypoints/s", "n_gpus": 1, "steps": served["frames"], "warmup": warm,
        "ms_per_step": span_ms / max(1, served["frames"]), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f16", "data": "synthetic",
        "config": {"workload": "serving: %d streams, Poisson U[20,30] Hz x%g, resolutions %s, U[150,1500] "
                               "keypoints, 31x31, 4 levels, FB 1 px, binary16 storage, %g s after %g s warm-up"
                               % (len(trace.streams), args.serve_rate_mult,
                                  "752x480 (literal reading)" if literal else "{640x480..1920x1080}", dur, warm)},
        "p50_frame_ms": served["p50_frame_ms"], "p99_frame_ms": served["p99_frame_ms"],
        "served": served, "capacity": capacity, "plain": plain,
    }


def run_pair(args):
    """Single pair: one 752x480 frame pair, 150 keypoints, 21x21, 3 levels,
    float32 storage; one step = both pyramids + tracking, plain launches."""
    import torch
    import synth
    import oracle
    from paper_2607_01757_amd import lk

    pr = synth.pair(args.seed, 752, 480, 150, 8.0, 2.0)
    ctx = lk.lk_context_create(0, 0)
    a = torch.from_numpy(pr.prev).cuda()
    b = torch.from_numpy(pr.next).cuda()
    pa = lk.lk_pyramid_create(ctx, 752, 480, 3, lk.LK_STORAGE_F32)
    pb = lk.lk_pyramid_create(ctx, 752, 480, 3, lk.LK_STORAGE_F32)
    pts = torch.from_numpy(pr.pts).cuda()
    prm = lk.make_params(21, 3, 30, 0.01, 1e-6, 0.0)
    out, st, res, _ = lk.outputs(150, 3)

    def step():
        lk.lk_build_pyramid(ctx, pa, a)
        lk.lk_build_pyramid(ctx, pb, b)
        lk.lk_track(ctx, pa, pb, pts, None, 150, prm, out, st, res, None)
    wall, per = time_steps(step, args.steps, args.warmup)
    g_pts, g_st = out.cpu().numpy(), st.cpu().numpy()
    r = oracle.track(pr.prev, pr.next, pr.pts, win=21, levels=3, min_eig=1e-6, nthreads=os.cpu_count() or 1)
    ok = (g_st == 0) & (r.status == 0)
    err = np.abs(g_pts[ok] - r.pts[ok]).max(axis=1)
    result = {
        "metric": "tracked keypoints/sec + p50/p99 frame latency (single pair, plain per-frame)",
        "value": 150 * args.steps / wall, "unit": "keypoints/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": wall / args.steps * 1e3, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "single pair 752x480, 150 keypoints, 21x21, 3 levels, 30 iterations, eps 0.01, "
                               "float32 storage; step = both pyramids + tracking"},
        "p50_frame_ms": percentile(per, 50), "p99_frame_ms": percentile(per, 99),
        "error_vs_fp64_oracle_px": {"max": float(err.max()), "p99": float(np.percentile(err, 99)),
                                    "points": int(ok.sum())},
        "status_agreement": float(np.mean(g_st == r.status)),
    }
    lk.lk_pyramid_destroy(pa)
    lk.lk_pyramid_destroy(pb)
    lk.lk_context_destroy(ctx)
    return result


def run_detect(args):
    """Shi-Tomasi detection over the next frames of the 64-stream batch: a
    fresh detection (no occupied points) and a top-up that keeps new corners
    away from each stream's first 100 tracked keypoints."""
    import torch
    from paper_2607_01757_amd import lk
    import oracle

    streams = make_streams(args.streams, args.seed)
    ctx = lk.lk_context_create(0, 0)
    imgs = [torch.from_numpy(s.next).cuda() for s in streams]
    px = sum(s.width * s.height for s in streams)
    det = lk.lk_detector_create(ctx, len(streams), px)
    cap = args.gftt_corners
    prm = lk.gftt_params(1, 30, cap, 0, 0.01)
    occ = [torch.from_numpy(np.ascontiguousarray(s.pts[:100])).cuda() for s in streams]
    outs = [torch.empty((cap, 2), dtype=torch.float32, device="cuda") for _ in streams]
    cnts = torch.empty((len(streams),), dtype=torch.int32, device="cuda")

    def frames(with_occ):
        return [{"img": im, "out_xy": o, "count": cnts[i:i + 1], **({"occupied": occ[i]} if with_occ else {})}
                for i, (im, o) in enumerate(zip(imgs, outs))]
    fresh, topup = frames(False), frames(True)
    res = {}
    for name, fr in (("fresh", fresh), ("topup", topup)):
        wall, per = time_steps(lambda: lk.lk_detect_corners(det, fr, prm), args.steps, args.warmup)
        res[name] = {"ms_per_step": wall / args.steps * 1e3, "frames_per_s": len(streams) * args.steps / wall,
                     "mpx_per_s": px * args.steps / wall / 1e6, "corners": int(cnts.sum().item())}
        log("%s: %.3f ms/step (%d frames)  %.0f frames/s  %d corners" %
            (name, res[name]["ms_per_step"], len(streams), res[name]["frames_per_s"], res[name]["corners"]))
    # latency of one frame alone (the 752x480 stream)
    k = next(i for i, s in enumerate(streams) if (s.width, s.height) == (752, 480))
    one = [fresh[k]]
    _, lat = time_steps(lambda: lk.lk_detect_corners(det, one, prm), args.steps, args.warmup)
    # exactness spot check on two frames
    lk.lk_detect_corners(det, fresh, prm)
    torch.cuda.synchronize()
    n = cnts.cpu().numpy()
    for i in (0, k):
        want = oracle.gftt(streams[i].next, r=1, quality=0.01, min_dist=30, max_corners=cap)
        got = outs[i][:n[i]].cpu().numpy()
        assert np.array_equal(got, want), "detector differs from the oracle on frame %d" % i
    # algorithmic operations per pixel (radius 1): Scharr pair 16, tensor
    # products 3, separable 3x3 sums 12, two integer tensor combinations 2,
    # NMS 8 compares: 41 integer operations.  The binary64 response (10 more)
    # is not counted: the walk forms it for a few candidates in a hundred
    # pixels only.  A share of the algorithm's operations, not the unit's
    # utilisation: the walk packs two 16-bit operations into many of its
    # instructions.  One op per lane per clock, 256 CUs x 4 SIMDs x 16 lanes x
    # 2.4 GHz = 39.3 T lane-ops/s (the fp32 vector peak / 4: no FMA pairs, no
    # packed pairs)
    ops = px * 41
    peak_lane_ops = PEAK_FP32_TFLOPS / 4
    t = res["fresh"]["ms_per_step"] * 1e-3
    result = {
        "metric": "corner detection frames/sec (batched, 64 streams)", "value": res["fresh"]["frames_per_s"],
        "unit": "frames/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": res["fresh"]["ms_per_step"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "i32+f64", "data": "synthetic",
        "config": {"workload": "Shi-Tomasi detection on the next frames of 64 streams {640x480..1920x1080}: "
                               "3x3 block, quality 0.01, min distance 30, up to %d corners per frame" % cap,
                   "streams": len(streams), "pixels_per_step": px},
        "topup": res["topup"], "p50_frame_ms": percentile(lat, 50), "p99_frame_ms": percentile(lat, 99),
        "roofline": {"bound": "alu", "kernel": "detection step (reset, peaks, compaction, buckets, selection)",
                     "achieved": ops / t / 1e12, "peak": peak_lane_ops, "unit": "T VALU lane-ops/s",
                     "frac": ops / t / 1e12 / peak_lane_ops, "traffic": detect_traffic()},
    }
    if not args.no_cpu_baseline:
        sample = streams[:8]
        t0 = time.perf_counter()
        for s_ in sample:
            oracle.gftt(s_.next, r=1, quality=0.01, min_dist=30, max_corners=cap)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": len(sample) / dt, "unit": "frames/s", "cores": 1, "kind": "oracle",
                                  "sample": "first 8 of the 64 frames, one thread, %.1f s" % dt}
    lk.lk_detector_destroy(det)
    lk.lk_context_destroy(ctx)
    return result


def run_frontend(args):
    """The front-end step of every camera rig after the tracker: track pools
    over 64 stereo (or mono) streams.  One step = pyramids of the left and
    right frames of every stream (one batched build) + one lifecycle step of
    every pool (temporal pass, carry-over, Shi-Tomasi top-up to the cap,
    cross-camera gate, new identities)."""
    import torch
    import synth
    from concurrent.futures import ThreadPoolExecutor
    from paper_2607_01757_amd import lk

    n_str, distinct, reps_per = args.streams, 16, 4
    cap = args.pool_cap
    stereo = not args.mono
    t0 = time.time()
    res = [synth.RESOLUTIONS[q % len(synth.RESOLUTIONS)] for q in range(distinct)]
    seqs = [synth.StereoSequence(100 + q, width=w, height=h, n_frames=1000) for q, (w, h) in enumerate(res)]
    span = 8                                   # frames each stream plays back and forth
    n_frames = span + reps_per - 1
    jobs = [(q, f, c) for q in range(distinct) for f in range(n_frames) for c in ((0, 1) if stereo else (0,))]
    with ThreadPoolExecutor(8) as ex:
        rendered = list(ex.map(lambda j: seqs[j[0]].frame(j[1], j[2]), jobs))
    dev = {j: torch.from_numpy(im).cuda() for j, im in zip(jobs, rendered)}
    log("frontend: %d sequences x %d frames rendered in %.1fs" % (distinct, n_frames, time.time() - t0))

    def frame_of(stream, step):            # back and forth over `span` frames, offset per replica
        p = step % (2 * span - 2)
        p = p if p < span else 2 * span - 2 - p
        return stream % distinct, p + stream // distinct

    ctx = lk.lk_context_create(0, 0)
    dims = [res[i % distinct] for i in range(n_str)]
    left = [[lk.lk_pyramid_create(ctx, w, h, 3, 0) for _ in range(2)] for (w, h) in dims]
    right = [lk.lk_pyramid_create(ctx, w, h, 3, 0) for (w, h) in dims] if stereo else None
    state = lk.pool_state(n_str, cap)
    pool = lk.lk_pool_create(ctx, n_str, cap, sum(w * h for w, h in dims), state)
    temporal = lk.make_params(21, 3, 30, 0.01, 1e-6, 0.0)
    stereo_prm = lk.make_params(21, 3, 30, 0.01, 1e-6, 1.0)
    det = lk.gftt_params(1, 20, cap, 8, 0.01)

    def step(k):
        pyrs, imgs, frames = [], [], []
        for i in range(n_str):
            q, f = frame_of(i, k)
            cur = left[i][k & 1]
            pyrs.append(cur)
            imgs.append(dev[(q, f, 0)])
            if stereo:
                pyrs.append(right[i])
                imgs.append(dev[(q, f, 1)])
            frames.append((i, left[i][(k - 1) & 1] if k > 0 else None, cur, right[i] if stereo else None))
        lk.lk_build_pyramids(ctx, pyrs, imgs)
        lk.lk_pool_step(pool, frames, temporal, stereo_prm, det)

    k = 0
    for _ in range(max(args.warmup, 3)):
        step(k)
        k += 1
    torch.cuda.synchronize()
    evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(args.steps)]
    tw = time.perf_counter()
    for a, b in evs:
        a.record()
        step(k)
        b.record()
        k += 1
    torch.cuda.synchronize()
    wall = time.perf_counter() - tw
    per = [a.elapsed_time(b) for a, b in evs]
    # pool statistics and tracked points per step (untimed, synchronised)
    prev_n = carried = cand = admitted = 0
    counts = []
    for _ in range(args.steps):
        step(k)
        k += 1
        st = state["stats"].cpu().numpy().astype(np.int64)
        prev_n += int(st[:, 0].sum()); carried += int(st[:, 1].sum())
        cand += int((st[:, 1] + st[:, 2]).sum()); admitted += int(st[:, 3].sum())
        counts.append(int(state["count"].sum().item()))
    tracked_per_step = (prev_n + (cand if stereo else 0)) / args.steps
    step_s = wall / args.steps
    result = {
        "metric": "front-end steps/sec with track pools (64 %s streams) + tracked keypoints/sec" % (
            "stereo" if stereo else "mono"),
        "value": n_str / step_s, "unit": "frames/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": step_s * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "frontend: %d %s streams (16 homography sequences {640x480..1920x1080}, 4 time "
                               "offsets each, played back and forth), pools of %d tracks: pyramids of every "
                               "frame + temporal LK, carry-over, Shi-Tomasi top-up (min distance 20), %sidentities;"
                               " 21x21, 3 levels" % (n_str, "stereo" if stereo else "mono", cap,
                                                     "cross-camera gate (FB 1 px), " if stereo else "")},
        "p50_step_ms": percentile(per, 50), "p99_step_ms": percentile(per, 99),
        "tracked_keypoints_per_s": tracked_per_step / step_s,
        "forward_rate": carried / max(prev_n, 1),
        "admitted_per_stream": admitted / args.steps / n_str,
        "new_candidates_per_stream": (cand - carried) / args.steps / n_str,
        "live_tracks_per_stream": float(np.mean(counts)) / n_str,
    }
    log("frontend: %.3f ms/step (p99 %.3f), %.3g tracked kp/s, forward rate %.4f, %.1f tracks per stream" %
        (step_s * 1e3, result["p99_step_ms"], result["tracked_keypoints_per_s"], result["forward_rate"],
         result["live_tracks_per_stream"]))
    lk.lk_pool_destroy(pool)
    for p in [p for pr in left for p in pr] + (right or []):
        lk.lk_pyramid_destroy(p)
    lk.lk_context_destroy(ctx)
    return result


def run_epipolar(args):
    """Epipolar check after LK (the geometric verification of temporal
    correspondences): 64 sets (one per camera stream) of 256 correspondences
    (the paper's keypoint cap), 512 eight-point hypotheses each, 1 px
    threshold, in one call."""
    import torch
    import synth
    import oracle.epipolar as E_or
    from paper_2607_01757_amd import lk

    n_sets, n, h = args.streams, args.epi_points, args.epi_hypotheses
    views = [synth.two_view(args.seed * 1000 + k, n, forward=(k % 4 == 0)) for k in range(n_sets)]
    samples = [synth.ransac_samples(args.seed * 1000 + k, n, h) for k in range(n_sets)]
    sets = []
    for tv, smp in zip(views, samples):
        sets.append({"p": torch.from_numpy(tv.p).cuda(), "q": torch.from_numpy(tv.q).cuda(),
                     "samples": torch.from_numpy(smp).cuda(), "intr": tv.intr,
                     "counts": torch.empty((h,), dtype=torch.int32, device="cuda"),
                     "inliers": torch.empty((n,), dtype=torch.uint8, device="cuda"),
                     "best": torch.empty((2,), dtype=torch.int32, device="cuda"),
                     "model": torch.empty((9,), dtype=torch.float64, device="cuda")})
    ctx = lk.lk_context_create(0, 0)
    wall, per = time_steps(lambda: lk.lk_epipolar_check(ctx, sets, 1.0), args.steps, args.warmup)
    t = time_block(lambda: lk.lk_epipolar_check(ctx, sets, 1.0), max(args.steps, 10), args.warmup)
    got = [int(d["best"][1].item()) for d in sets]
    truth = [int((~tv.outlier).sum()) for tv in views]
    # algorithmic binary64 flops: per hypothesis the elimination of the 8 x 9
    # system (sum over pivots of 2 (8-k)(9-k) plus back substitution, ~580),
    # the pixel-space model (~60), and 21 per scored correspondence
    flops = n_sets * h * (640 + 21 * n)
    step = wall / args.steps
    result = {
        "metric": "epipolar checks/sec (batched, 64 sets of 256 correspondences x 512 hypotheses)",
        "value": n_sets / step, "unit": "sets/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": step * 1e3, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64", "data": "synthetic",
        "config": {"workload": "epipolar: %d sets of %d two-view correspondences (20%% outliers, 0.3 px noise, every "
                               "4th set forward motion), %d eight-point hypotheses each, 1 px threshold" % (
                                   n_sets, n, h)},
        "p50_step_ms": percentile(per, 50), "p99_step_ms": percentile(per, 99),
        "hypothesis_scores_per_s": n_sets * h * n / t,
        "inliers_found_vs_planted": float(np.mean(np.array(got) / np.array(truth))),
        "roofline": {"bound": "alu", "kernel": "k_epi_hypotheses+k_epi_best", "achieved": flops / t / 1e12,
                     "peak": 78.6, "unit": "TFLOP/s (fp64 vector)", "frac": flops / t / 1e12 / 78.6, "traffic": None},
    }
    if not args.no_cpu_baseline:
        k = min(n_sets, 64)
        t0 = time.perf_counter()
        for tv, smp in list(zip(views, samples))[:k]:
            E_or.check(tv.p, tv.q, smp, tv.intr, 1.0)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": k / dt, "unit": "sets/s", "cores": 1, "kind": "oracle",
                                  "sample": "first %d of the %d sets, numpy on one thread, %.1f s" % (k, n_sets, dt)}
    log("epipolar: %.3f ms per call (%d sets), %.3g sets/s, best inliers / planted %.3f" %
        (step * 1e3, n_sets, n_sets / step, result["inliers_found_vs_planted"]))
    lk.lk_context_destroy(ctx)
    return result


SWEEP_KP = (160, 192, 256, 384, 512, 768, 1000, 1500)


def run_sweep(args):
    """Tracker cost against the keypoint budget per frame and the frame size
    (the paper's keypoint-count ablation and its observation that front-end
    time grows with the pixel count; Sec. IV).  For every resolution of the
    batched workload and every budget: 64 streams of that shape in one tuned,
    graph-captured step (pyramids + tracking), the tracker alone, and one
    frame alone through the plain per-frame calls."""
    import torch
    import synth
    from paper_2607_01757_amd import lk

    ctx = lk.lk_context_create(0, 0)
    n_str = args.streams
    distinct = min(n_str, 8)          # distinct frame pairs per resolution, repeated over the streams
    reps = max(args.steps, 10)
    rows = []
    for (w, h) in synth.RESOLUTIONS:
        t0 = time.time()
        base = [synth.pair(args.seed * 1000 + s, w, h, max(SWEEP_KP)) for s in range(distinct)]
        streams = [base[s % distinct] for s in range(n_str)]
        wl = BatchedWorkload(lk, ctx, streams)
        t_pyr = wl.time_build(reps, args.warmup)
        log("%dx%d: %d streams ready in %.1fs, pyramids %.3f ms" % (w, h, n_str, time.time() - t0, t_pyr * 1e3))
        for kp in SWEEP_KP:
            n = kp * n_str
            pts = torch.from_numpy(np.concatenate([s.pts[:kp] for s in streams])).cuda()
            pairs = [(a, b, i * kp, kp) for i, (a, b) in enumerate(zip(wl.prev_pyr, wl.next_pyr))]
            out, st, res, _ = lk.outputs(n, 3)
            step, best, _ = prepared_step(lk, ctx, wl.next_pyr, wl.next_img, pairs, pts, wl.params, out, st, res)
            trk = lk.lk_batch_create(ctx, [], [], pairs, pts, None, wl.params, out, st, res, None,
                                     config=lk.lk_exec_config(best.persistent, best.blocks_per_cu, 0, best.chunk,
                                                      best.waves_per_group, 0))
            t_trk = time_block(lambda: lk.lk_batch_run(trk), reps, args.warmup)
            t_step = time_block(lambda: lk.lk_batch_run(step), reps, args.warmup)

            def plain():
                lk.lk_build_pyramid(ctx, wl.next_pyr[0], wl.next_img[0])
                lk.lk_track(ctx, wl.prev_pyr[0], wl.next_pyr[0], pts[:kp], None, kp, wl.params, out[:kp],
                            st[:kp], res[:kp], None)
            t_plain = time_block(plain, reps, args.warmup)
            lat = []
            for _ in range(reps):       # one frame alone: events around it, idle GPU before
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record(); plain(); b.record()
                torch.cuda.synchronize()
                lat.append(a.elapsed_time(b))
            ok = float((st == 0).float().mean().item())
            rows.append({"width": w, "height": h, "kp_per_frame": kp, "streams": n_str, "keypoints": n,
                         "step_ms": t_step * 1e3, "tracker_ms": t_trk * 1e3, "pyramid_ms": t_pyr * 1e3,
                         "kp_per_s": n / t_step, "tracker_kp_per_s": n / t_trk,
                         "tracker_ns_per_kp": t_trk / n * 1e9, "plain_frame_ms": t_plain * 1e3,
                         "plain_frame_latency_p50_ms": percentile(lat, 50),
                         "exec": [best.persistent, best.blocks_per_cu], "tracked_fraction": ok})
            log("  %4d kp/frame: step %.3f ms (%.3g kp/s), tracker %.3f ms (%.2f ns/kp), plain frame %.3f ms "
                "back to back, %.3f ms alone" % (kp, t_step * 1e3, n / t_step, t_trk * 1e3, t_trk / n * 1e9,
                                                 t_plain * 1e3, percentile(lat, 50)))
            lk.lk_batch_destroy(step)
            lk.lk_batch_destroy(trk)
            del pts, out, st, res
        wl.close()
        del wl
        torch.cuda.synchronize()
    # normalised to the 256-keypoint budget at each resolution (the paper's
    # presentation of its ablation)
    ref = {(r["width"], r["height"]): r for r in rows if r["kp_per_frame"] == 256}
    for r in rows:
        b = ref[(r["width"], r["height"])]
        r["plain_frame_rel_256"] = r["plain_frame_latency_p50_ms"] / b["plain_frame_latency_p50_ms"]
        r["step_rel_256"] = r["step_ms"] / b["step_ms"]
    big = max(rows, key=lambda r: (r["width"] * r["height"], r["kp_per_frame"]))
    lk.lk_context_destroy(ctx)
    return {
        "metric": "tracked keypoints/sec against keypoints per frame and frame size (batched, 64 streams)",
        "value": big["kp_per_s"], "unit": "keypoints/s", "n_gpus": 1, "steps": reps, "warmup": args.warmup,
        "ms_per_step": big["step_ms"], "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "sweep: %d streams of one resolution in {640x480..1920x1080} x keypoints per "
                               "frame in %s; 21x21, 3 levels, 30 iterations, eps 0.01, float32 storage; value = "
                               "the 1920x1080, %d-keypoint point" % (n_str, list(SWEEP_KP), max(SWEEP_KP))},
        "rows": rows,
    }


def run_copy(args):
    """Plain device copy of a known size (calibrates rocprof byte counters)."""
    import torch
    n = 256 << 20
    a = torch.empty(n, dtype=torch.uint8, device="cuda").fill_(1)
    b = torch.empty_like(a)
    for _ in range(3):
        b.copy_(a)
    torch.cuda.synchronize()
    return {"metric": "device copy", "bytes_read": n, "bytes_written": n, "launches": 3}


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--workload", default="batched", choices=["batched", "pair", "stereo", "stereo16", "serve",
                                                           "detect", "sweep", "frontend", "epipolar", "copy"])
    ap.add_argument("--frames", type=int, default=1000, help="stereo workloads: sequence length")
    ap.add_argument("--precision-frames", type=int, default=-1,
                    help="stereo workloads: frames compared with the FP64 oracle (-1: all, 0: none)")
    ap.add_argument("--gain-mode", choices=["smooth", "iid"], default="smooth",
                    help="stereo workloads: exposure drifting smoothly in [0.9, 1.1], or drawn per frame")
    ap.add_argument("--serve-streams", type=int, default=256)
    ap.add_argument("--serve-seconds", type=float, default=10.0)
    ap.add_argument("--serve-warmup", type=float, default=2.0)
    ap.add_argument("--serve-inflight", type=int, default=2)
    ap.add_argument("--serve-threads", type=int, default=8, help="submitter threads of the serve workload")
    ap.add_argument("--serve-rate-mult", type=float, default=1.0, help="arrival-rate multiplier (serve workload)")
    ap.add_argument("--serve-res", choices=["mixed", "literal"], default="mixed",
                    help="serve workload resolutions: the batched set, or every stream 752x480")
    ap.add_argument("--streams", type=int, default=64)
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--cpu-streams", type=int, default=64)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-plain", action="store_true")
    ap.add_argument("--gftt-corners", type=int, default=200)
    ap.add_argument("--pool-cap", type=int, default=256, help="tracks per stream (frontend workload)")
    ap.add_argument("--mono", action="store_true", help="frontend workload without the cross-camera gate")
    ap.add_argument("--epi-points", type=int, default=256, help="correspondences per set (epipolar workload)")
    ap.add_argument("--epi-hypotheses", type=int, default=512, help="hypotheses per set (epipolar workload)")
    ap.add_argument("--storage", choices=["f32", "f16"], default="f32",
                    help="pyramid storage of the batched workload")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (streams would be sharded "
              "across GPUs with no exchange); run with --gpus 1", file=sys.stderr)
        sys.exit(2)
    if args.workload == "copy":
        res = run_copy(args)
    elif args.workload == "serve":
        res = run_serve(args)
    elif args.workload == "detect":
        res = run_detect(args)
    elif args.workload == "sweep":
        res = run_sweep(args)
    elif args.workload == "frontend":
        res = run_frontend(args)
    elif args.workload == "epipolar":
        res = run_epipolar(args)
    elif args.workload == "pair":
        res = run_pair(args)
    elif args.workload in ("stereo", "stereo16"):
        res = run_stereo(args, args.workload == "stereo16")
    else:
        res = run_batched(args)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
