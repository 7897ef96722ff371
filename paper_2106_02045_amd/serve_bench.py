"""Serving benchmark: a stream of camera frames with Poisson arrivals.

    python -m paper_2106_02045_amd.serve_bench [--frames 100000] [--fps 1000]

Each frame carries U{20..200} fiducial spots (ROI side in {9, 13, 17, 21},
symmetric Gaussian, sigma U[1.5, 2.5], amplitude U[1000, 5000], background 150,
Poisson noise).  The C++ replay driver submits every frame at its scheduled
arrival time; the serving loop admits frames by device memory, folds all
admitted frames into the next launch and overlaps launches on several streams.
Per-frame latency = arrival -> results in the caller's host arrays.  Prints one
JSON line with p50 / p99 latency and sustained fits/s, and checks that frames
fitted in the mix give the same bits as the same spots fitted alone.

--track M: instead, every frame holds the same M markers (13x13 ROIs) of a
drifting sample (random walk plus sway), and the loop tracks the drift on the
device (spotfit_serve_track, window --window frames); the line then also gives
the tracked drift's error against the true drift.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def main(argv=None):
    print(json.dumps(run(argv)))


def run(argv=None) -> dict:
    """Run the serving benchmark with command-line style arguments; returns the
    record that main() prints."""
    ap = argparse.ArgumentParser()
    ap.add_argument("--frames", type=int, default=20000)
    ap.add_argument("--fps", type=float, default=1000.0)
    ap.add_argument("--streams", type=int, default=2)
    ap.add_argument("--budget-mb", type=int, default=256)
    ap.add_argument("--max-frames", type=int, default=8192)
    ap.add_argument("--schedule", default="mixed", choices=["mixed", "uniform"])
    ap.add_argument("--check", type=int, default=200, help="frames compared with a direct fit")
    ap.add_argument("--seed", type=int, default=4)
    ap.add_argument("--plan", default="latency", choices=["latency", "throughput"],
                    help="plan hint of the fit (latency: never another mapping than the default one)")
    ap.add_argument("--device-init", action="store_true",
                    help="frames carry no start values: the loop computes them on the device")
    ap.add_argument("--track", type=int, default=0, help="markers per frame of a tracked sample")
    ap.add_argument("--window", type=int, default=16, help="frames in the tracked drift mean")
    ap.add_argument("--warmup-frames", type=int, default=200,
                    help="frames replayed through a throw-away server first, so that the "
                         "timed replay does not include the first launch of each kernel "
                         "(code-object loading) or the first use of the streams")
    a = ap.parse_args(argv)

    import torch

    import paper_2106_02045_amd as sf
    import spotgen

    t0 = time.time()
    if a.track > 0:
        ref, truth_drift, frames = spotgen.drift_frames(a.frames, n_markers=a.track, side=13,
                                                        fps=a.fps, seed=a.seed)
        gaps = np.random.default_rng(a.seed).exponential(1.0 / a.fps, size=a.frames)
        arrivals = np.cumsum(gaps)
    else:
        arrivals, frames = spotgen.serve_frames(a.frames, fps=a.fps, seed=a.seed, threads=16)
    gen_s = time.time() - t0
    opts = sf.default_options(max_side=21, schedule=(sf.SCHEDULE_MIXED if a.schedule == "mixed"
                                                     else sf.SCHEDULE_UNIFORM),
                              plan_hint=(sf.PLAN_LATENCY if a.plan == "latency" else sf.PLAN_THROUGHPUT))
    if a.warmup_frames > 0:
        m = min(a.warmup_frames, len(frames))
        warm = sf.Server(0, opts, device_mem_budget=a.budget_mb << 20, max_frames=a.max_frames,
                         n_streams=a.streams)
        warm.replay([(f.data, f.sizes, None if a.device_init else f.init, False)
                     for f in frames[:m]],
                    np.round((arrivals[:m] - arrivals[0]) * 1e9).astype(np.uint64))
        warm.close()
    srv = sf.Server(0, opts, device_mem_budget=a.budget_mb << 20, max_frames=a.max_frames,
                    n_streams=a.streams)
    if a.track > 0:
        srv.track(ref, a.window)
    offs = np.round((arrivals - arrivals[0]) * 1e9).astype(np.uint64)
    w0 = time.perf_counter()
    outs = srv.replay([(f.data, f.sizes, None if a.device_init else f.init, a.track > 0)
                       for f in frames], offs)
    wall = time.perf_counter() - w0
    st = srv.stats()
    srv.close()

    # the same spots fitted alone, directly: identical bits
    dev = torch.device("cuda:0")
    ctx = sf.Context(0)
    rng = np.random.default_rng(a.seed)
    check = np.sort(rng.choice(len(frames), size=min(a.check, len(frames)), replace=False))
    mismatched = 0
    for f in check:
        b = frames[f]
        up = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev)
        d = (up(b.data), up(b.sizes), up(b.offsets))
        g = ctx.fit_raw(*d, opts) if a.device_init else ctx.fit_spots(*d, up(b.init), opts)
        torch.cuda.synchronize()
        same = (np.array_equal(g["params"].cpu().numpy(), outs[f]["params"]) and
                np.array_equal(g["status"].cpu().numpy(), outs[f]["status"]) and
                np.array_equal(g["iters"].cpu().numpy(), outs[f]["iters"]))
        mismatched += int(not same)

    spots = int(sum(f.n for f in frames))
    tracking = None
    if a.track > 0:
        got = np.concatenate([o["drift"] for o in outs])
        W = a.window
        tw = np.stack([truth_drift[max(0, f - W + 1):f + 1].mean(axis=0) for f in range(len(frames))])
        mean_err = np.stack([got["mean_dx"], got["mean_dy"]], axis=1) - tw
        frame_err = np.stack([got["dx"], got["dy"]], axis=1) - truth_drift
        tracking = {"markers": a.track, "window": W,
                    "rms_frame_drift_error_px": float(np.sqrt(np.nanmean(frame_err ** 2))),
                    "rms_tracked_drift_error_px": float(np.sqrt(np.nanmean(mean_err[W:] ** 2))),
                    "drift_range_px": float(np.ptp(truth_drift)),
                    "frames_without_marker": int((got["n_used"] == 0).sum())}
    rec = {
        "metric": "p99 frame latency",
        "value": st["latency_p99_us"],
        "unit": "us",
        "higher_is_better": False,
        "latency_p50_us": st["latency_p50_us"],
        "latency_p99_us": st["latency_p99_us"],
        "latency_max_us": st["latency_max_us"],
        "fits_per_s": spots / st["wall_s"] if st["wall_s"] > 0 else None,
        "frames": a.frames,
        "spots": spots,
        "fps_offered": a.fps,
        "fps_achieved": a.frames / st["wall_s"] if st["wall_s"] > 0 else None,
        "wall_s": st["wall_s"],
        "batches": st["batches"],
        "mean_frames_per_batch": st["mean_frames_per_batch"],
        "rejected_submits": st["rejected"],
        "frames_failed": st["frames_failed"],
        "streams": a.streams,
        "budget_mb": a.budget_mb,
        "schedule": a.schedule,
        "start_values": "device" if a.device_init else "host",
        "plan": a.plan,
        "alone_vs_mix": {"frames_checked": int(len(check)), "frames_differing": mismatched},
        "tracking": tracking,
        "data": "synthetic",
        "config": ({"workload": "drift_markers", "frames": a.frames, "fps": a.fps,
                    "spots_per_frame": a.track, "roi_sides": [13]} if a.track > 0 else
                   {"workload": "serve_fiducials", "frames": a.frames, "fps": a.fps,
                    "spots_per_frame": "U{20..200}", "roi_sides": [9, 13, 17, 21]}),
        "warmup_frames": a.warmup_frames,
        "gen_s": gen_s,
    }
    return rec


if __name__ == "__main__":
    main()
