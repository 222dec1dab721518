#!/usr/bin/env python3
"""Benchmark: foveated Mpix/s on 1920x1080 RGB u8 frames, one MI355X.

One step = one 1080p RGB frame foveated by foveate_forward (plan, weights,
tile staging, horizontal pass, vertical pass, u8 epilogue and foveal copies
all run inside the one kernel launch).  Step k reads and writes frame k mod
pool of a pool resident in HBM (96 frames, about 1.2 GB of inputs and
outputs by default) and draws a fresh fixation uniformly from the central
half; the JSON line states how many pool frames and bytes the timed steps
touched (fewer than the pool when there are fewer steps than frames).

Prints one JSON line.  `roofline` prices the forward kernel's algorithmic
FP32 FMA work (halo-inclusive separable count, foveal fragments zero) against
the chip's FP32 vector peak; `cpu_baseline` times the FP64 oracle on a bounded
sample of the same workload.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import re
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "foveated Mpix/s (1080p RGB) + p99 frame latency, served vs plain launch"
PROFILE_EVERY = 4  # main-kernel timing samples one call in four of the timed region
H, W, C = 1080, 1920, 3
PEAK_FP32_TFLOPS = 157.3  # MI355X FP32 vector, published (two wave64 FMA instructions issued per SIMD every four cycles)
HBM_PEAK_GBS = 8000.0


def algorithmic_fma(h, w, c, p, plan_r):
    """FP32 FMAs of the separable method for one frame: per fragment and
    channel N*bw*(bh+2r) (horizontal pass over the padded rows) + N*bw*bh
    (vertical pass); foveal fragments (r = 0) cost none."""
    B = p["block"]
    nby, nbx = plan_r.shape
    total = 0
    for by in range(nby):
        y0 = max(p["origin_y"] + by * B, 0)
        bh = min(p["origin_y"] + (by + 1) * B, h) - y0
        for bx in range(nbx):
            r = int(plan_r[by, bx])
            if r == 0:
                continue
            x0 = max(p["origin_x"] + bx * B, 0)
            bw = min(p["origin_x"] + (bx + 1) * B, w) - x0
            n = 2 * r + 1
            total += c * (n * bw * (bh + 2 * r) + n * bw * bh)
    return total


KERNEL_SOURCES = ("paper_2012_08655_amd/csrc/forward.hip", "paper_2012_08655_amd/csrc/forward.h",
                  "paper_2012_08655_amd/csrc/conv.h", "paper_2012_08655_amd/csrc/common.h",
                  "paper_2012_08655_amd/csrc/fixed.h", "paper_2012_08655_amd/csrc/order.h")
TRAFFIC_SUMMARY = os.path.join(ROOT, "profiles", "fov_fwd_u8_1080p_rgb_traffic.md")


def kernel_source_hash():
    h = hashlib.sha256()
    for rel in KERNEL_SOURCES:
        with open(os.path.join(ROOT, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic():
    """HBM bytes per launch of the forward kernel from the committed
    rocprofv3 PMC summary (FETCH_SIZE + WRITE_SIZE, scaled by the copy-kernel
    calibration), or None when the summary is missing or the kernel sources
    changed since the counters were taken."""
    try:
        text = open(TRAFFIC_SUMMARY).read()
    except OSError:
        return None
    vals = dict(re.findall(r"^- (\w+): ([0-9a-f.]+)\s*$", text, re.M))
    if vals.get("kernel_source_hash") != kernel_source_hash():
        return None
    try:
        return float(vals["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def copy_calibration(mb, reps):
    """A plain device-to-device copy of a known size, for scaling the PMC
    byte counters (profile it with --pmc FETCH_SIZE / WRITE_SIZE)."""
    import torch
    n = mb * (1 << 20)
    src = torch.ones(n, dtype=torch.uint8, device="cuda:0")
    dst = torch.empty_like(src)
    for _ in range(reps):
        dst.copy_(src)
    torch.cuda.synchronize()
    print(json.dumps({"copy_calibration_bytes_per_dispatch": n, "reps": reps}))


def cpu_baseline(frame, rng_seed=99, target_s=10.0):
    """FP64 oracle (all host threads) on whole frames of the same workload
    (fresh central-half fixation per frame) until target_s seconds of CPU work
    have run; the last frame may be a random pixel subset to bound the time."""
    import oracle
    import synth
    oracle.build(force=False)
    x = frame.transpose(2, 0, 1).astype(np.float64)
    rng = np.random.default_rng(rng_seed)
    done_px, spent, frames = 0, 0.0, 0
    while spent < target_s:
        p = synth.params_cfg2(rng)
        left = target_s - spent
        per_px = spent / done_px if done_px else None
        if per_px is None:
            npts = 100000  # calibration sample
        else:
            npts = H * W if per_px * H * W <= left else max(1000, int(left / per_px))
        ys, xs = np.divmod(rng.permutation(H * W)[:npts], W)
        t0 = time.perf_counter()
        oracle.forward_points(x, p, ys, xs)
        spent += time.perf_counter() - t0
        done_px += npts
        frames += 1
    return {"value": done_px / spent / 1e6, "unit": "Mpix/s", "cores": oracle.max_threads(), "kind": "oracle",
            "sample": "%d pixels (x3 channels) over %d 1920x1080 RGB frames with random central-half fixations, "
                      "FP64 direct 2-D, %.1f s" % (done_px, frames, spent)}


def _spin_until(lib, target):
    while lib.foveate_now() < target:
        pass


def serving_leg(rates, seconds, warm_s, budget_mib, max_batch, use_graph=True, seed=4, ring=8, inflight=4,
                shared_stream=False):
    """Open-loop Poisson request traces (16 viewer sessions of mixed
    resolution, saccade + drift gaze) replayed twice on the same GPU: once
    through the continuous-batching server, once as plain per-frame
    foveate_forward calls on one stream.  Latency = completion seen on the
    host minus the scheduled arrival; frames arriving in the first warm_s
    seconds are excluded."""
    import ctypes
    import torch
    import synth
    from paper_2012_08655_amd import _native as N, api
    from paper_2012_08655_amd.server import Server

    lib = N.lib()
    dev = torch.device("cuda:0")
    inputs = {}
    for k, (h, w) in enumerate(synth.frames.RESOLUTIONS):
        inputs[(h, w)] = torch.from_numpy(synth.grating_frame(h, w, 3, seed=20 + k)).to(dev)
    in_desc = {key: api.tensor_desc(t, "HWC") for key, t in inputs.items()}
    stream = torch.cuda.Stream(device=dev)
    sh = ctypes.c_void_p(stream.cuda_stream)
    legs = []
    for ri, rate in enumerate(rates):
        tr = synth.poisson_trace(rate, warm_s + seconds, seed=seed + ri)
        n = len(tr["t"])
        outs, out_desc = {}, {}
        din, dout, prm = [], [], []
        count = {}
        for i in range(n):
            s, key = int(tr["session"][i]), (int(tr["h"][i]), int(tr["w"][i]))
            if s not in outs:
                outs[s] = [torch.empty_like(inputs[key]) for _ in range(ring)]
                out_desc[s] = [api.tensor_desc(o, "HWC") for o in outs[s]]
            k = count.get(s, 0)
            count[s] = k + 1
            din.append(in_desc[key])
            dout.append(out_desc[s][k % ring])
            prm.append(N.make_params(synth.params_dict(tr["fix_x"][i], tr["fix_y"][i], 64.0, tr["slope"][i], 16.0)))
        pixels = tr["h"] * tr["w"]
        measured = tr["t"] >= warm_s
        max_frag = max_batch * 8160  # 16 x 4K frames of 32x32 fragments
        res = {"offered_fps": rate, "frames": int(measured.sum()),
               "mean_mpix_per_frame": round(float(pixels[measured].mean()) / 1e6, 3)}
        for mode in ("plain", "served"):
            torch.cuda.synchronize()
            done = np.zeros(n)
            launched = np.zeros(n)
            batch = np.zeros(n, np.int32)
            if mode == "plain":
                stamps = (ctypes.c_double * n)()
                dptr = ctypes.POINTER(ctypes.c_double)
                slots = [ctypes.cast(ctypes.addressof(stamps) + 8 * i, dptr) for i in range(n)]
                t0 = lib.foveate_now() + 0.02
                for i in range(n):
                    _spin_until(lib, t0 + tr["t"][i])
                    N.check(lib.foveate_forward(ctypes.byref(din[i]), ctypes.byref(dout[i]), ctypes.byref(prm[i]),
                                                1, sh))
                    N.check(lib.foveate_stream_timestamp(sh, slots[i]))
                stream.synchronize()
                deadline = time.time() + 10
                while stamps[n - 1] == 0.0 and time.time() < deadline:
                    time.sleep(0.001)
                done[:] = np.frombuffer(stamps, dtype=np.float64)
                batch[:] = 1
            else:
                srv = Server(hbm_budget_bytes=budget_mib << 20, max_batch_frames=max_batch, max_inflight_batches=inflight,
                             max_requests=8192, max_fragments=max_frag, max_sigma=16.0, use_graph=use_graph,
                             shared_stream=shared_stream)
                tickets = np.zeros(n, np.uint64)
                tk = ctypes.c_uint64()
                done_flag = ctypes.c_int32()
                tm = N.FovTiming()
                oldest = 0

                def retire(i):
                    N.check(lib.foveate_poll(srv._h, ctypes.c_uint64(int(tickets[i])), ctypes.byref(done_flag),
                                             ctypes.byref(tm)))
                    if done_flag.value:
                        done[i] = tm.t_done
                        launched[i] = tm.t_launch
                        batch[i] = tm.batch_frames
                    return bool(done_flag.value)

                t0 = lib.foveate_now() + 0.02
                for i in range(n):
                    _spin_until(lib, t0 + tr["t"][i])
                    N.check(lib.foveate_submit(srv._h, ctypes.byref(din[i]), ctypes.byref(dout[i]),
                                               ctypes.byref(prm[i]), None, ctypes.byref(tk)))
                    tickets[i] = tk.value
                    while oldest < i and retire(oldest):
                        oldest += 1
                srv.drain()
                for i in range(oldest, n):
                    if not retire(i):
                        raise RuntimeError("served frame %d not done after drain" % i)
                srv.close()
            lat = (done - (t0 + tr["t"]))[measured] * 1e3
            span = done[measured].max() - (t0 + tr["t"][measured].min())
            res[mode] = {"p50_ms": round(float(np.percentile(lat, 50)), 4),
                         "p99_ms": round(float(np.percentile(lat, 99)), 4),
                         "max_ms": round(float(lat.max()), 4),
                         "mpix_s": round(float(pixels[measured].sum()) / span / 1e6, 1),
                         "mean_batch_frames": round(float(batch[measured].mean()), 3)}
            if mode == "served":
                # where the served latency goes: arrival -> launch (admission, batching, host
                # launch work) and launch -> completion seen by the host
                wait = (launched - (t0 + tr["t"]))[measured] * 1e3
                run = (done - launched)[measured] * 1e3
                res[mode]["to_launch_p50_p99_ms"] = [round(float(np.percentile(wait, q)), 4) for q in (50, 99)]
                res[mode]["launch_to_done_p50_p99_ms"] = [round(float(np.percentile(run, q)), 4) for q in (50, 99)]
            print("bench: serving %s at %g fps: p50 %.3f ms, p99 %.3f ms" % (mode, rate, res[mode]["p50_ms"],
                                                                          res[mode]["p99_ms"]),
                  file=sys.stderr, flush=True)
        legs.append(res)
        del outs
    return {"budget_mib": budget_mib, "max_batch_frames": max_batch, "max_inflight_batches": inflight,
            "shared_stream": shared_stream, "sessions": 16,
            "seconds_measured": seconds, "warmup_s": warm_s, "hip_graph": use_graph,
            "latency": "host-seen completion minus scheduled arrival",
            "plain": "one foveate_forward per frame on one stream at its arrival time",
            "rates": legs}


def _time_calls(fn, reps, stream):
    """Median and p99 milliseconds of fn() over reps calls (HIP events on stream)."""
    import torch
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(reps)]
    for a, b in ev:
        a.record(stream)
        fn()
        b.record(stream)
    torch.cuda.synchronize()
    ms = np.array([a.elapsed_time(b) for a, b in ev])
    return float(np.median(ms)), float(np.percentile(ms, 99))


def batch_leg(reps=10, seed=11):
    """64 frames of mixed resolution (640x480 .. 3840x2160 RGB u8, per-frame
    central-half fixation and slope in [0.01, 0.04]) in one autotuned launch,
    against the same frames as 64 plain per-frame launches."""
    import torch
    import synth
    import paper_2012_08655_amd as fov
    dev = torch.device("cuda:0")
    frames, params = synth.batch_mixed(64, seed=seed, unique_content=1)
    ins = [torch.from_numpy(f).to(dev) for f in frames]
    outs = [torch.empty_like(t) for t in ins]
    stream = torch.cuda.current_stream()
    mpix = sum(f.shape[0] * f.shape[1] for f in frames) / 1e6
    tuned = fov.autotune_batch(ins, params, outs, layout="HWC", reps=3)
    fov.forward_batch(ins, params, outs, layout="HWC")
    med_b, p99_b = _time_calls(lambda: fov.forward_batch(ins, params, outs, layout="HWC"), reps, stream)

    def plain():
        for t, o, p in zip(ins, outs, params):
            fov.forward(t, p, out=o, layout="HWC")

    plain()
    med_p, p99_p = _time_calls(plain, reps, stream)
    return {"frames": 64, "mpix_per_batch": round(mpix, 2), "launch_config": tuned,
            "batched": {"ms_median": round(med_b, 4), "ms_p99": round(p99_b, 4), "mpix_s": round(mpix / med_b * 1e3, 1)},
            "plain_per_frame": {"ms_median": round(med_p, 4), "ms_p99": round(p99_p, 4),
                                "mpix_s": round(mpix / med_p * 1e3, 1)}}


def host_pipeline_leg(frames=300, depth=4, distinct=8, seed=13):
    """End-to-end rate with the frames in pinned host memory (the paper's
    165 Hz includes its transfers), through the library's host pipeline
    (foveate_pipeline_*): per frame an upload, the foveation and a download,
    overlapped across `depth` device slots.  `distinct` different pinned
    frames are cycled, each step with its own central-half fixation."""
    import torch
    import synth
    from paper_2012_08655_amd.pipeline import HostPipeline
    rng = np.random.default_rng(seed)
    host_in = [torch.from_numpy(synth.grating_frame(H, W, C, seed=seed + k)).pin_memory() for k in range(distinct)]
    nbuf = depth + 1
    host_out = [torch.empty_like(host_in[0]).pin_memory() for _ in range(nbuf)]
    params = [synth.params_cfg2(rng) for _ in range(frames + 2 * depth)]
    with HostPipeline(H * W * C, depth=depth) as pl:

        def run(n, first):
            tickets = []
            for i in range(n):
                if i >= depth:
                    pl.wait(tickets[i - depth])  # at most `depth` frames in flight
                tickets.append(pl.submit(host_in[i % distinct], params[first + i], out=host_out[i % nbuf]))
            for t in tickets[max(0, n - depth):]:
                pl.wait(t)

        run(2 * depth, 0)
        t0 = time.perf_counter()
        run(frames, 2 * depth)
        wall = time.perf_counter() - t0
    return {"frames": frames, "pipeline_depth": depth, "distinct_frames": distinct, "fps": round(frames / wall, 1),
            "ms_per_frame": round(wall * 1e3 / frames, 4), "mpix_s": round(frames * H * W / wall / 1e6, 1),
            "transfer": "pinned host u8 HWC 1920x1080x3 in and out; upload, foveation and download on three "
                        "streams of the library's host pipeline",
            "paper_context": "165 Hz on a GTX 1060 including transfers"}


def adjoint_leg(reps=20, seed=12):
    """Forward and adjoint (foveate_backward) on training-style batches:
    32 x 3x224x224 and 4 x 3x512x512 float32, fixation uniform over the image,
    slope 0.03, cap 12, e0 32."""
    import torch
    import synth
    import paper_2012_08655_amd as fov
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream()
    rng = np.random.default_rng(seed)
    out = []
    for n, s in ((32, 224), (4, 512)):
        x = torch.from_numpy(synth.uniform_frames((n, 3, s, s), seed=seed + s)).to(dev)
        ps = [synth.params_cfg5(rng, s, s) for _ in range(n)]
        y = fov.forward(x, ps)
        g = torch.empty_like(y)
        fov.backward(y, ps, grad_in=g)
        fwd_ms, _ = _time_calls(lambda: fov.forward(x, ps, out=y), reps, stream)
        adj_ms, _ = _time_calls(lambda: fov.backward(y, ps, grad_in=g), reps, stream)
        mpix = n * s * s / 1e6
        out.append({"batch": "%dx3x%dx%d f32" % (n, s, s), "forward_ms": round(fwd_ms, 4),
                    "adjoint_ms": round(adj_ms, 4), "forward_mpix_s": round(mpix / fwd_ms * 1e3, 1),
                    "adjoint_mpix_s": round(mpix / adj_ms * 1e3, 1)})
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=400)
    ap.add_argument("--warmup", type=int, default=40)
    ap.add_argument("--pool", type=int, default=96, help="frames resident in HBM")
    ap.add_argument("--distinct", type=int, default=4, help="distinct frame contents in the pool")
    ap.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    ap.add_argument("--cpu-seconds", type=float, default=10.0)
    ap.add_argument("--serve-rates", default="120,480,1920", help="offered frames/s of the serving traces")
    ap.add_argument("--serve-seconds", type=float, default=10.0, help="measured seconds per serving trace")
    ap.add_argument("--serve-budget-mib", type=int, default=256)
    ap.add_argument("--serve-max-batch", type=int, default=16)
    ap.add_argument("--serve-graph", type=int, default=1, help="1: the server replays captured hipGraphs")
    ap.add_argument("--serve-inflight", type=int, default=4, help="batches the server keeps in flight")
    ap.add_argument("--serve-shared-stream", type=int, default=0,
                    help="1: in-flight batches queue on one stream instead of one stream each")
    ap.add_argument("--no-serve", action="store_true", help="skip the serving traces")
    ap.add_argument("--no-extra", action="store_true", help="skip the batch and adjoint legs")
    ap.add_argument("--no-autotune", action="store_true", help="time the default launch configuration")
    ap.add_argument("--batch-only", action="store_true",
                    help="only run the 64-frame mixed batch leg (for a kernel trace) and exit")
    ap.add_argument("--adjoint-only", action="store_true",
                    help="only run the forward/adjoint leg on the training batches (for a kernel trace) and exit")
    ap.add_argument("--copy-calibration", type=int, default=0, metavar="MB",
                    help="only run a plain MB-sized device copy (counter calibration) and exit")
    args = ap.parse_args()
    if args.copy_calibration:
        copy_calibration(args.copy_calibration, 5)
        return
    if args.batch_only:
        import paper_2012_08655_amd as fov
        fov.load()
        print(json.dumps({"batch": batch_leg()}))
        return
    if args.adjoint_only:
        import paper_2012_08655_amd as fov
        fov.load()
        print(json.dumps({"adjoint": adjoint_leg()}))
        return
    if args.gpus != 1:
        print("bench.py measures one GPU only: the method needs no communication and this build "
              "runs on a single MI355X (frames shard trivially across GPUs)", file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2012_08655_amd as fov
    import synth

    fov.load()
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    print("bench: building frame pool", file=sys.stderr, flush=True)
    distinct = [synth.grating_frame(H, W, C, seed=1 + i) for i in range(args.distinct)]
    pool_in = torch.empty((args.pool, H, W, C), dtype=torch.uint8, device=dev)
    for i in range(args.pool):
        pool_in[i].copy_(torch.from_numpy(distinct[i % args.distinct]))
    pool_out = torch.empty_like(pool_in)
    rng = np.random.default_rng(1)
    nsteps = args.warmup + args.steps
    params = [synth.params_cfg2(rng) for _ in range(nsteps)]
    stream = torch.cuda.current_stream()

    def step(i):
        k = i % args.pool
        fov.forward(pool_in[k], params[i], out=pool_out[k], layout="HWC", stream=stream)

    tuned = None
    if not args.no_autotune:
        # untimed: pick the launch configuration for this workload class
        print("bench: autotune", file=sys.stderr, flush=True)
        tuned = fov.autotune(pool_in[0], params[0], out=pool_out[0], layout="HWC", reps=5, stream=stream)
    print("bench: warmup", file=sys.stderr, flush=True)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()

    # Timed region: exactly `steps` frames.  The library times the main kernel
    # of one call in PROFILE_EVERY with HIP
    # events that the kernel's own dispatch stamps on the launch stream (a
    # stamped dispatch does not overlap the next kernel, so the other calls
    # run without events).
    nprof = (args.steps + PROFILE_EVERY - 1) // PROFILE_EVERY
    fov.profile_begin(nprof, every=PROFILE_EVERY)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for j in range(args.steps):
        step(args.warmup + j)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kms = fov.profile_end(nprof)
    assert len(kms) == nprof
    # Device time of whole calls, untimed: torch
    # events around each call put marker packets between calls.
    nlat = min(args.steps, 200)
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(nlat)]
    for j in range(nlat):
        ev[j][0].record(stream)
        step(args.warmup + j)
        ev[j][1].record(stream)
    torch.cuda.synchronize()
    call_ms = np.array([a.elapsed_time(b) for a, b in ev])
    print("bench: timed %d steps in %.3f s" % (args.steps, wall), file=sys.stderr, flush=True)

    mpix = H * W / 1e6
    value = args.steps * mpix / wall
    # roofline of the forward kernel: algorithmic FLOPs per launch / mean launch time
    fmas = []
    for j in range(0, args.steps, PROFILE_EVERY):  # the profiled calls
        p = params[args.warmup + j]
        _, r = fov.plan_host(H, W, p)
        fmas.append(algorithmic_fma(H, W, C, p, r))
    flops = 2.0 * np.array(fmas, dtype=np.float64)
    achieved_tflops = float(np.mean(flops / (kms * 1e-3)) / 1e12)
    bytes_per_frame = H * W * C * 2
    achieved_gbs = float(bytes_per_frame / (kms.mean() * 1e-3) / 1e9)
    traffic = measured_traffic()

    result = {
        "metric": METRIC,
        "value": round(value, 1),
        "unit": "Mpix/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(wall * 1e3 / args.steps, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic: 1920x1080 RGB u8 gratings + noise, %d-frame HBM pool, fixation uniform in central half" % args.pool,
        "pool": {"frames": args.pool, "distinct_contents": args.distinct,
                 "frames_touched_by_timed_steps": min(args.steps, args.pool),
                 "bytes_touched_by_timed_steps": min(args.steps, args.pool) * H * W * C * 2},
        "config": {"workload": "1920x1080 RGB u8 -> u8, 32x32 fragments, sigma = 0.02*(e-64) capped at 16, "
                               "radius ceil(3 sigma), clamp-to-edge, one frame per launch",
                   "frame_pixels": H * W, "channels": C, "block": 32},
        "frame_latency_ms": {"p50": round(float(np.percentile(call_ms, 50)), 5),
                             "p99": round(float(np.percentile(call_ms, 99)), 5),
                             "kind": "plain per-frame launch: device time of one call, HIP events"},
        "roofline": {"bound": "alu", "kernel": "fov_fwd_u8_kernel",
                     "note": "8-bit output in fixed point on the integer matrix cores, byte for byte the FP32 sums; "
                             "algorithmic FP32 operations against the FP32 vector peak",
                     "achieved": round(achieved_tflops, 3), "peak": PEAK_FP32_TFLOPS, "unit": "TFLOP/s",
                     "frac": round(achieved_tflops / PEAK_FP32_TFLOPS, 4), "traffic": traffic,
                     "algorithmic_flops_per_launch": float(np.mean(flops)),
                     "mean_launch_ms": round(float(kms.mean()), 5),
                     "timed_launches": "%d of %d (one in %d)" % (len(kms), args.steps, PROFILE_EVERY),
                     "hbm_GBs_algorithmic": round(achieved_gbs, 1)},
        "launch_config": tuned or "default (split 1, 64 strip rows, one workgroup per work item)",
        "paper_context": "GTX 1060: 1.65 ms kernel for one 1920x1080 RGB frame (~1257 Mpix/s), 165 Hz with transfers",
    }
    if not args.no_extra:
        print("bench: batch leg", file=sys.stderr, flush=True)
        result["batch"] = batch_leg()
        print("bench: adjoint leg", file=sys.stderr, flush=True)
        result["adjoint"] = adjoint_leg()
        print("bench: host pipeline leg", file=sys.stderr, flush=True)
        result["host_pipeline"] = host_pipeline_leg()
    if not args.no_serve:
        rates = [float(r) for r in args.serve_rates.split(",") if r]
        result["serving"] = serving_leg(rates, args.serve_seconds, 0.5, args.serve_budget_mib, args.serve_max_batch,
                                        use_graph=bool(args.serve_graph), inflight=args.serve_inflight,
                                        shared_stream=bool(args.serve_shared_stream))
    if not args.no_cpu:
        print("bench: cpu baseline", file=sys.stderr, flush=True)
        result["cpu_baseline"] = cpu_baseline(distinct[0], target_s=args.cpu_seconds)
    print(json.dumps(result))


if __name__ == "__main__":
    main()
