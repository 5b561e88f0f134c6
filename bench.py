#!/usr/bin/env python3
"""Benchmark of the integer Winograd F(4x4,3x3) layer with tap-wise
power-of-two quantization on one MI355X.

One step = one pass of the whole online path over one batch: input transform
with tap-wise requant (K1) and the 36-tap int8 MFMA GEMM with the fused
output transform, bias and requant (K2), i.e. one wino_f4_conv_int8 call (small
layers: one launch for both).  Inputs are resident in HBM before the timed region.  The default workload is
the largest layer (N=4, 256->256, 160x160, NHWC), the configuration the
tap-GEMM MFMA-utilisation target refers to.

Printed on one JSON line: the contract fields, the roofline of the dominant
kernel (durations from HIP events on the launch stream), the kernels'
figures, the direct int8 convolution of the same library on the same layer
(speed-up), and the CPU oracle timed on a bounded sample.
"""
import argparse
import dataclasses
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "Winograd F4 int8 conv: effective TOPS (direct-equiv) + % of int8 MFMA peak"
PEAK_INT8_TOPS = 5000.0      # MI355X dense int8 MFMA, TOP/s
PEAK_FP16_TFLOPS = 2500.0    # MI355X dense fp16 MFMA, TFLOP/s (the int8/10 tap GEMM)
PEAK_HBM_GBS = 8000.0        # MI355X HBM3E, GB/s


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--config", default="C5", help="C1 .. C5")
    ap.add_argument("--layer", type=int, default=0,
                    help="layer of a chained configuration (C3: 0..3); layers after the first get "
                         "an input drawn with the configuration's activation recipe at their shape")
    ap.add_argument("--layout", default="nhwc", choices=["nchw", "nhwc"])
    ap.add_argument("--variant", default="split", choices=["split", "fused"])
    ap.add_argument("--transform", default="f4", choices=["f4", "f2"],
                    help="Winograd F(4x4,3x3) (the default) or F(2x2,3x3)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--bits", type=int, default=8, choices=[8, 10],
                    help="Winograd-domain integer width: 8, or 10 for the int8/10 variant")
    ap.add_argument("--tap-kernel", default="auto",
                    choices=["auto", "resident", "rows", "rows_streamk", "waves", "64x32", "32x32", "16x16"],
                    help="force the tap-GEMM kernel (wino_f4_plan_set_tap_kernel)")
    ap.add_argument("--no-direct", action="store_true")
    ap.add_argument("--no-plan-timing", action="store_true", help="skip timing the on-device plan builds")
    ap.add_argument("--cpu-images", type=int, default=0,
                    help="oracle sample size in images; 0 = as many as fill ~10 s of CPU work")
    ap.add_argument("--chain", action="store_true",
                    help="C3 only: time the four layers as one chained step (each layer's input the previous "
                         "layer's GPU output, 2x2 max-pooled where the stage halves the image), eager and as a "
                         "replayed HIP graph, with the algorithm wino_select_algorithm picks per layer")
    ap.add_argument("--share-batch", type=int, default=0,
                    help="one GPU's share of a batch-sharded layer: the first N images of the workload")
    ap.add_argument("--share-cout", type=int, default=0,
                    help="one GPU's share of an output-channel-sharded layer: the first C output channels")
    ap.add_argument("--copy-probe", action="store_true",
                    help="also run a plain 256 MiB device-to-device copy (scale reference for HBM counters)")
    return ap.parse_args()


def counter_traffic(cfg, layout, kernel, transform="f4"):
    """HBM bytes per launch of `kernel` from the committed rocprofv3 counter
    summary (FETCH_SIZE and WRITE_SIZE, each scaled by what the counter
    reads for a plain copy of known size), or None when there is no
    summary for this workload or the kernel source changed since the
    counters were taken."""
    import hashlib
    tag = cfg if transform == "f4" else f"{cfg}_{transform}"
    path = os.path.join(ROOT, "profiles", f"{tag}_{layout}_hbm_counters.txt")
    if not os.path.exists(path):
        return None
    vals, kern = {}, {}
    for line in open(path):
        tok = line.split()
        if not tok or tok[0].startswith("#"):
            continue
        if tok[0] == "source_sha256":
            vals["src_file"], vals["src_hash"] = tok[1], tok[2]
        elif tok[0] == "kernel":
            kern[tok[1]] = (float(tok[3]), float(tok[5]))
        elif len(tok) == 2:
            vals[tok[0]] = float(tok[1])
    # the hash covers every listed source ("a.hip+b.h": the files' bytes in order)
    h = hashlib.sha256()
    for name in vals.get("src_file", "").split("+"):
        src = os.path.join(ROOT, "paper_2209_12982_amd", "csrc", name)
        if not name or not os.path.isfile(src):
            return None
        h.update(open(src, "rb").read())
    if h.hexdigest() != vals.get("src_hash"):
        return None
    for name, (f, w) in kern.items():
        if name.startswith(kernel):
            return f * 1024 * vals["fetch_scale"] + w * 1024 * vals["write_scale"]
    return None


def check_output(torch, y, layout, args, share, layer=None):
    """SHA-256 of the timed step's output (NCHW order) against the oracle's
    record for this configuration and layer in tests/golden (written by
    tests/golden/make_golden.py from the oracle alone).  True / False, or
    None where no record applies (a GPU's share of a layer, the C3 layers
    past the first, whose inputs are the previous layer's outputs, F2 at
    10 bits)."""
    import hashlib
    if layer is None:
        layer = args.layer
        if args.config == "C3" and layer > 0:
            return None
    if share or (args.transform != "f4" and args.bits != 8):
        return None
    path = os.path.join(ROOT, "tests", "golden", "configs.json" if args.bits == 8 else "configs_i10.json")
    if not os.path.exists(path):
        return None
    key = "layers" if args.transform == "f4" else "f2_layers"
    rec = json.load(open(path)).get(args.config, {}).get(key, [])
    if len(rec) <= layer or "sha256_nchw" not in rec[layer]:
        return None
    torch.cuda.synchronize()
    yn = y.cpu().numpy()
    if layout == 1:   # NHWC -> NCHW
        yn = yn.transpose(0, 3, 1, 2)
    import numpy as np
    digest = hashlib.sha256(np.ascontiguousarray(yn).tobytes()).hexdigest()
    return digest == rec[layer]["sha256_nchw"]


def time_loop(torch, fn, steps):
    """Average ms per call over `steps` back-to-back calls, HIP events on the
    current stream (the stream every library call is enqueued on)."""
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    s.record()
    for _ in range(steps):
        fn()
    e.record()
    torch.cuda.synchronize()
    return s.elapsed_time(e) / steps


def time_calls(torch, fn, calls):
    """Per-call GPU duration: an event pair on the launch stream around each
    call, so host-side call overhead between calls is not counted (it is for
    short kernels in a back-to-back loop).  Returns (median, p10, p90) ms."""
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(calls)]
    torch.cuda.synchronize()
    for s, e in ev:
        s.record()
        fn()
        e.record()
    torch.cuda.synchronize()
    t = sorted(s.elapsed_time(e) for s, e in ev)
    q = lambda f: t[min(len(t) - 1, int(f * (len(t) - 1) + 0.5))]
    return q(0.5), q(0.1), q(0.9)


def time_cold(torch, fn, calls, flush):
    """Per-call GPU duration with the device caches flushed before each call:
    a 1 GiB buffer is read between calls (a sum over it), which evicts the
    call's inputs from L2 and from the 256 MB Infinity Cache (MALL) and
    leaves clean lines there, so the call reads its inputs from HBM and
    pays no write-back of someone else's data.  As in kernel_ms, the smaller
    of two estimates: the median of event pairs around single calls (which
    also count the dispatch latency after the flush) and the difference
    between a loop of flush + call and a loop of flushes alone, divided by
    the calls.  Returns (ms, p10, p90) with p10/p90 of the event pairs."""
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(calls)]
    torch.cuda.synchronize()
    for s, e in ev:
        flush.sum()
        s.record()
        fn()
        e.record()
    torch.cuda.synchronize()
    t = sorted(s.elapsed_time(e) for s, e in ev)
    q = lambda f: t[min(len(t) - 1, int(f * (len(t) - 1) + 0.5))]

    def loop(with_call):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        s.record()
        for _ in range(calls):
            flush.sum()
            if with_call:
                fn()
        e.record()
        torch.cuda.synchronize()
        return s.elapsed_time(e)
    diff = (loop(True) - loop(False)) / calls
    return (min(q(0.5), diff) if diff > 0 else q(0.5)), q(0.1), q(0.9)


def kernel_ms(torch, fn, calls):
    """A single-kernel call's duration: the smaller of the back-to-back loop
    average (exact for long kernels, host-bound for short ones) and the
    per-call event-pair median (exact for short kernels, plus the events' own
    overhead for long ones); with the per-call p10 and p90."""
    med, p10, p90 = time_calls(torch, fn, calls)
    return min(med, time_loop(torch, fn, calls)), p10, p90


def cpu_baseline(x, layers_plan, n_img, spec, layers_plan_f, target_s=10.0):
    """The oracle's online path (a-1 .. a-6, plan excluded) on images of the
    same workload, one at a time and cycling through the batch: n_img images
    if n_img > 0, else as many as fill target_s seconds of CPU work."""
    import numpy as np
    from oracle import tapwise
    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        threads = 1
    n = x.shape[0]
    done, dt = 0, 0.0
    while (done < n_img) if n_img > 0 else (dt < target_s):
        xs = np.ascontiguousarray(x[done % n:done % n + 1])
        t0 = time.perf_counter()
        tapwise.conv_int8(xs, layers_plan)
        dt += time.perf_counter() - t0
        done += 1
    ops = 2.0 * 9 * done * spec.h * spec.w * spec.cin * spec.cout
    # the oracle's direct int8 convolution on the same images, a shorter sample
    from oracle import direct
    wq, _ = direct.quantize_weights_pow2(layers_plan_f)
    ddone, ddt = 0, 0.0
    while ddt < target_s / 4:
        xs = np.ascontiguousarray(x[ddone % n:ddone % n + 1])
        t0 = time.perf_counter()
        direct.conv_int8(xs, wq, None, 8, False)
        ddt += time.perf_counter() - t0
        ddone += 1
    dops = 2.0 * 9 * ddone * spec.h * spec.w * spec.cin * spec.cout
    return {"value": ops / dt / 1e12, "unit": "TOPS", "cores": int(threads), "kind": "oracle",
            "direct_int8": {"value": dops / ddt / 1e12, "unit": "TOPS",
                            "sample": f"{ddone} single-image passes of the oracle's direct int8 convolution "
                                      f"(numpy int64), {ddt:.2f} s"},
            "sample": f"{done} single-image passes cycling over the {n} images of the same layer, full online "
                      f"path (numpy int64 transforms, float64 BLAS tap GEMM), {dt:.2f} s",
            "seconds": dt, "host_cpus": os.cpu_count(),
            "affinity": len(os.sched_getaffinity(0)) if hasattr(os, "sched_getaffinity") else None}


def run_chain(args):
    """The C3 stack as one step: four layers chained on the device, NHWC.
    Per layer, wino_select_algorithm picks direct, F2 or F4 (direct is not
    chained here: a layer that picks it runs F2, and the line says so);
    calibration and plans are set up untimed on the layer's real chained
    input.  Between stages the 2x2 max-pooling is two elementwise maxima
    (glue of the workload, not part of a layer; timed on its own)."""
    import numpy as np
    import torch

    import paper_2209_12982_amd as W
    import workloads

    torch.cuda.set_device(0)
    wl = workloads.WORKLOADS["C3"]
    x, layers = workloads.generate("C3")
    n = x.shape[0]
    cur = torch.from_numpy(np.ascontiguousarray(x.transpose(0, 2, 3, 1))).cuda()
    stages, ops, picked = [], 0.0, []
    for k, (f, bias, spec) in enumerate(layers):
        pool = None
        if k > 0 and (spec.h, spec.w) != (layers[k - 1][2].h, layers[k - 1][2].w):
            # rows first (two contiguous half-images), then column pairs
            rows = cur.view(n, spec.h, 2, 2 * spec.w * spec.cin)
            t = torch.empty((n, spec.h, 2 * spec.w * spec.cin), dtype=torch.int8, device="cuda")
            cols = t.view(n, spec.h, spec.w, 2, spec.cin)
            dst = torch.empty((n, spec.h, spec.w, spec.cin), dtype=torch.int8, device="cuda")

            def pool(rows=rows, t=t, cols=cols, dst=dst):
                torch.maximum(rows[:, :, 0], rows[:, :, 1], out=t)
                torch.maximum(cols[:, :, :, 0], cols[:, :, :, 1], out=dst)
            pool()
            cur = dst
        algo = W.wino_select_algorithm(n, spec.cin, spec.cout, spec.h, spec.w, W.NHWC)
        mt = 4 if algo == W.ALGO_F4 else 2
        picked.append({W.ALGO_F4: "f4", W.ALGO_F2: "f2", W.ALGO_DIRECT: "direct (ran f2)"}[algo])
        calibrate = W.wino_f4_calibrate_input if mt == 4 else W.wino_f2_calibrate_input
        make_plan = W.wino_f4_plan if mt == 4 else W.wino_f2_plan
        eb, _ = calibrate(cur, n, spec.cin, spec.h, spec.w, W.NHWC)
        plan0 = make_plan(f, eb, bias=bias, out_shift=0, relu=spec.relu)
        ws = torch.empty(max(1, W.wino_f4_workspace_bytes(plan0, n, spec.h, spec.w)), dtype=torch.int8,
                         device="cuda")
        s, _ = W.wino_f4_calibrate_output(plan0, cur, n, spec.h, spec.w, W.NHWC, ws)
        plan = make_plan(f, eb, bias=bias, out_shift=s, relu=spec.relu)
        y = torch.empty((n, spec.h, spec.w, spec.cout), dtype=torch.int8, device="cuda")
        stages.append((pool, plan, cur, y, ws, spec))
        W.wino_f4_conv_int8(plan, cur, y, n, spec.h, spec.w, W.NHWC, W.SPLIT, ws)
        cur = y
        ops += 2.0 * 9 * n * spec.h * spec.w * spec.cin * spec.cout
    torch.cuda.synchronize()

    def step():
        for pool, plan, xin, y, ws, spec in stages:
            if pool is not None:
                pool()
            W.wino_f4_conv_int8(plan, xin, y, n, spec.h, spec.w, W.NHWC, W.SPLIT, ws)

    # per-layer and pooling times first: they also bring the clocks up before
    # the timed steps (as in the single-layer bench)
    layer_ms = []
    for pool, plan, xin, y, ws, spec in stages:
        layer_ms.append(kernel_ms(torch, lambda plan=plan, xin=xin, y=y, ws=ws, spec=spec: W.wino_f4_conv_int8(
            plan, xin, y, n, spec.h, spec.w, W.NHWC, W.SPLIT, ws), max(args.steps, 50))[0])
    pools = [st[0] for st in stages if st[0] is not None]
    pool_ms = sum(kernel_ms(torch, p, max(args.steps, 50))[0] for p in pools)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    eager_ref = stages[-1][3].clone()
    ms = time_loop(torch, step, args.steps)
    # every layer's output of the timed chain against the oracle's F4 chain
    # (records exist for F4 only: a chain where a layer runs F2 is not checked)
    bitexact = None
    if all(p == "f4" for p in picked):
        bitexact = all(check_output(torch, st[3], W.NHWC, args, None, layer=k) for k, st in enumerate(stages))

    # the same step captured once as a HIP graph and replayed: the launches
    # of the step's kernels are submitted as one graph launch
    g = torch.cuda.CUDAGraph()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        step()
    torch.cuda.current_stream().wait_stream(s)
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        step()
    replays_ok = True
    for _ in range(3):
        stages[-1][3].zero_()
        g.replay()
        torch.cuda.synchronize()
        replays_ok &= bool(torch.equal(stages[-1][3], eager_ref))
    graph_ms = time_loop(torch, g.replay, args.steps)

    line = {
        "metric": METRIC, "value": ops / (ms * 1e-3) / 1e12, "unit": "TOPS", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "int8", "data": "synthetic",
        "config": {"workload": f"C3 chain: {wl.desc}, four layers chained on the device", "n": n,
                   "layout": "nhwc", "algorithms": picked,
                   "layers": [f"{sp.cin}->{sp.cout}@{sp.h}x{sp.w}" for _, _, _, _, _, sp in stages]},
        "layer_ms": layer_ms, "pool_ms": pool_ms,
        "graph": {"ms_per_step": graph_ms, "TOPS": ops / (graph_ms * 1e-3) / 1e12,
                  "replays_match_eager": replays_ok},
        "roofline": None, "cpu_baseline": None, "bitexact": bitexact,
    }
    print(json.dumps(line), flush=True)
    if bitexact is False:
        sys.exit("bench: the timed chain's output differs from the oracle's golden record")


def main():
    args = parse()
    if args.gpus != 1:
        print(f"bench.py measures one GPU; --gpus {args.gpus} is not supported "
              "(the layer shards by batch with no communication between GPUs)", file=sys.stderr)
        sys.exit(2)
    if args.chain:
        if args.config != "C3":
            print("--chain times the C3 stack; use --config C3", file=sys.stderr)
            sys.exit(2)
        return run_chain(args)
    import numpy as np
    import torch

    import paper_2209_12982_amd as W
    import workloads

    torch.cuda.set_device(0)
    layout = W.NHWC if args.layout == "nhwc" else W.NCHW
    variant = W.SPLIT if args.variant == "split" else W.FUSED
    wl = workloads.WORKLOADS[args.config]
    x, layers = workloads.generate(args.config)
    f, bias, spec = layers[args.layer]
    if args.layer > 0:
        x = workloads.draw_activations(np.random.default_rng(1000 + args.layer), (x.shape[0], spec.cin, spec.h, spec.w),
                                       wl.act, wl.zero_frac)
    share = None
    if args.share_batch > 0:
        # batch sharding: every GPU runs its images with the whole plan
        x = np.ascontiguousarray(x[:args.share_batch])
        share = f"images 0..{x.shape[0] - 1} of {wl.n} (batch split)"
    if args.share_cout > 0:
        # output-channel sharding: every GPU holds the plan of its channels
        # and reads the whole input
        f, bias = f[:args.share_cout], bias[:args.share_cout]
        spec = dataclasses.replace(spec, cout=f.shape[0])
        share = (share + "; " if share else "") + f"output channels 0..{f.shape[0] - 1} (channel split)"
    n, cin, cout, h, w = x.shape[0], spec.cin, spec.cout, spec.h, spec.w
    xa = x if layout == W.NCHW else np.ascontiguousarray(x.transpose(0, 2, 3, 1))
    xd = torch.from_numpy(xa).cuda()
    yshape = (n, cout, h, w) if layout == W.NCHW else (n, h, w, cout)
    y = torch.empty(yshape, dtype=torch.int8, device="cuda")

    # offline: calibration and plan (not timed)
    mt = 4 if args.transform == "f4" else 2
    if args.bits == 10:
        calibrate = W.wino_f4_calibrate_input_i10 if mt == 4 else W.wino_f2_calibrate_input_i10
        make_plan = W.wino_f4_plan_i10 if mt == 4 else W.wino_f2_plan_i10
    else:
        calibrate = W.wino_f4_calibrate_input if mt == 4 else W.wino_f2_calibrate_input
        make_plan = W.wino_f4_plan if mt == 4 else W.wino_f2_plan
    eb, _ = calibrate(xd, n, cin, h, w, layout)
    plan0 = make_plan(f, eb, bias=bias, out_shift=0, relu=spec.relu)
    ws = torch.empty(max(1, W.wino_f4_workspace_bytes(plan0, n, h, w, W.SPLIT)), dtype=torch.int8, device="cuda")
    out_shift = spec.out_shift
    if out_shift is None:
        out_shift, _ = W.wino_f4_calibrate_output(plan0, xd, n, h, w, layout, ws)
    t0 = time.perf_counter()
    plan = make_plan(f, eb, bias=bias, out_shift=out_shift, relu=spec.relu)
    plan_host_ms = (time.perf_counter() - t0) * 1e3
    info = W.wino_f4_plan_info(plan)
    W.wino_f4_plan_set_tap_kernel(plan, {"auto": W.TAP_AUTO, "resident": W.TAP_RESIDENT, "rows": W.TAP_ROWS,
                                         "rows_streamk": W.TAP_ROWS_STREAMK, "waves": W.TAP_WAVES, "64x32": W.TAP_RESIDENT_64X32,
                                         "32x32": W.TAP_RESIDENT_32X32,
                                         "16x16": W.TAP_RESIDENT_16X16}[args.tap_kernel])
    plan_ms = {"host_exact": plan_host_ms}
    if not args.no_plan_timing and args.bits == 8:
        # the same plan with the weight transform on the device: fp32 weights,
        # and int8 spatial weights (one power-of-two scale); wall time of the
        # whole call (allocation, kernels, read-back, synchronization), median
        make_dev = W.wino_f4_plan_device if mt == 4 else W.wino_f2_plan_device
        make_i8 = W.wino_f4_plan_int8 if mt == 4 else W.wino_f2_plan_int8
        fd = torch.from_numpy(np.ascontiguousarray(f, dtype=np.float32)).cuda()
        wq8, e_f = W.direct_conv_quantize_weights(f)
        wi8 = torch.from_numpy(np.ascontiguousarray(wq8.transpose(0, 3, 1, 2))).cuda()
        torch.cuda.synchronize()
        for key, mk in (("device_fp32", lambda: make_dev(fd, eb, bias=bias, out_shift=out_shift, relu=spec.relu)),
                        ("device_int8", lambda: make_i8(wi8, e_f, eb, bias=bias, out_shift=out_shift,
                                                        relu=spec.relu))):
            ts = []
            for _ in range(5):
                t0 = time.perf_counter()
                pd = mk()
                ts.append((time.perf_counter() - t0) * 1e3)
                if key == "device_fp32":
                    di = W.wino_f4_plan_info(pd)
                    assert di["e_g"] == info["e_g"] and di["sh"] == info["sh"], "device plan differs"
                pd.close()
            plan_ms[key] = float(np.median(ts))

    def step():
        W.wino_f4_conv_int8(plan, xd, y, n, h, w, layout, variant, ws if variant == W.SPLIT else None)

    # per-kernel durations: each of the two launches of a step timed on its
    # own (HIP events on the launch stream), see kernel_ms; where the step is
    # one launch, that one, and the two launches beside it as another route
    th, tw = (h + mt - 1) // mt, (w + mt - 1) // mt
    T = n * th * tw
    ntap = (mt + 2) ** 2
    lay = 1 if layout == W.NHWC else 0
    kern = W.wino_probe_conv_kernels(plan, xd, n, h, w, layout)
    one_launch = variant == W.SPLIT and kern["launches"] == 1
    # the two launches of the split calls: an odd address never takes the one launch
    two = W.wino_probe_conv_kernels(plan, 1, n, h, w, layout) if one_launch else kern
    # kernel names as the profiler shows them (template arguments included; the
    # tap-resident kernel's block configuration is a class argument).
    # the one-instruction requantization serves plans whose e_B are all <= 16 - bits
    sat = "true" if all(0 <= e <= 16 - args.bits for e in eb) else "false"
    if layout == W.NHWC and cin >= 4:
        # tiles per block: 8 unless 16 leaves fewer idle tiles per row
        k1_tx = 8 if (-tw) % 8 <= (-tw) % 16 else 16
        k1_name, k1_inst = "wino_input_xform_nhwc", f"wino_input_xform_nhwc<{mt},{args.bits},{k1_tx},{sat}>"
    else:
        k1_name, k1_inst = "wino_input_xform", f"wino_input_xform<{mt},{lay},{args.bits},{two['xform_tiles']},{sat}>"
    gemm = two["gemm"]
    if gemm == "rows_wide":
        k2_name = "wino_tap_gemm_rows_wide"
        k2_inst = f"wino_tap_gemm_rows_wide<{lay},10,{'int' if info['epilogue_bits'] == 32 else 'longlong'}>"
    elif gemm == "rows_streamk":
        k2_name, k2_inst = "wino_tap_gemm_rows_sk", f"wino_tap_gemm_rows_sk<{lay}>"
    elif gemm == "rows":
        cfg = "32,3,4" if two["tiles"] == 32 else "64,6,3"
        k2_name, k2_inst = "wino_tap_gemm_rows", f"wino_tap_gemm_rows<RwCfg<{cfg}>,{lay},{'true' if cin <= 64 else 'false'},0>"
    elif gemm == "waves":
        # 64-channel chunks per ring stage: the largest of 4, 3, 2, 1 dividing the padded chunks
        nkc = (cin + 63) // 64
        nk = next(k for k in (4, 3, 2, 1) if nkc % k == 0)
        k2_name, k2_inst = "wino_tap_gemm_ws", f"wino_tap_gemm_ws<{lay}, {nk}>"
    elif gemm == "small":
        k2_name = "wino_tap_gemm_small"
        k2_inst = f"wino_tap_gemm_small<{mt},{two['co'] // 16},{two['tiles'] // 16},{lay},0>"
    else:
        k2_name, k2_inst = "wino_tap_gemm", f"wino_tap_gemm<{mt},{lay},{info['epilogue_bits']},0,{args.bits}>"
    cs_name, cs_inst = "wino_conv_small", f"wino_conv_small<{mt},{kern['co'] // 16},{lay},{sat}>"
    k1_ms = k2_ms = None
    if variant == W.SPLIT:
        k1 = lambda: W.wino_f4_input_transform(plan, xd, n, h, w, layout, ws)
        k2 = lambda: W.wino_f4_tap_gemm(plan, ws, y, n, h, w, layout)
        k1_ms, k1_p10, k1_p90 = kernel_ms(torch, k1, max(args.steps, 50))
        k2_ms, k2_p10, k2_p90 = kernel_ms(torch, k2, max(args.steps, 50))
        if one_launch:
            cs_ms, cs_p10, cs_p90 = kernel_ms(torch, step, max(args.steps, 50))

    # the timed steps: W warmup steps, then exactly K steps back to back.  They
    # run after the per-kernel timings, which keep the GPU busy for a few ms
    # first: straight after the untimed setup (host-side plan builds, idle
    # GPU) the first milliseconds of steps run 5-12% slower while the clocks
    # come up, which is not the steady-state rate of a loop of layers
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    ms = time_loop(torch, step, args.steps)
    bitexact = check_output(torch, y, layout, args, share)

    # cold: every call starts with its inputs in HBM only (caches flushed)
    flush = torch.ones(1 << 27, dtype=torch.int64, device="cuda")
    ncold = max(5, min(20, args.steps))
    cold = {"step_ms": time_cold(torch, step, ncold, flush)[0]}
    if variant == W.SPLIT:
        cold["kernels_ms"] = {k1_name: time_cold(torch, k1, ncold, flush)[0],
                              k2_name: time_cold(torch, k2, ncold, flush)[0]}
    del flush

    direct_ops = 2.0 * 9 * n * h * w * cin * cout
    tap_ops = 2.0 * ntap * T * cin * cout
    # the int8/10 tap GEMM multiplies exact 10-bit integers on fp16 matrix cores
    k2_peak, k2_unit = (PEAK_FP16_TFLOPS, "TFLOP/s") if args.bits == 10 else (PEAK_INT8_TOPS, "TOP/s")
    value = direct_ops / (ms * 1e-3) / 1e12
    eb_bytes = 2 if args.bits == 10 else 1                       # Vq / Uq element: int8 or fp16
    k1_bytes = n * h * w * cin + eb_bytes * ntap * T * cin      # read x, write Vq
    k2_bytes = eb_bytes * (ntap * T * cin + ntap * cin * cout) + n * h * w * cout + 4 * cout
    # the whole layer against the HBM roofline: the bytes any implementation
    # must move (x, y, Uq, bias) and the SPLIT path's extra Vq round trip
    fused_min = n * h * w * cin + n * h * w * cout + eb_bytes * ntap * cin * cout + 4 * cout
    split_bytes = fused_min + 2 * eb_bytes * ntap * T * cin
    layer_hbm = {"alg_bytes_min": fused_min, "frac_min": fused_min / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS}
    if not one_launch:                                          # no Vq in memory in the one launch
        layer_hbm.update({"alg_bytes_split": split_bytes, "GB/s_split": split_bytes / (ms * 1e-3) / 1e9,
                          "frac_split": split_bytes / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS})
    kernels, two_launches = {}, None
    cfg_tag = args.config + (f"L{args.layer}" if args.layer else "") + ("_i10" if args.bits == 10 else "")
    if k1_ms is not None:
        kernels[k1_name] = {"ms": k1_ms, "p10_ms": k1_p10, "p90_ms": k1_p90, "bound": "hbm", "bytes": k1_bytes,
                            "GB/s": k1_bytes / (k1_ms * 1e-3) / 1e9,
                            "frac": k1_bytes / (k1_ms * 1e-3) / 1e9 / PEAK_HBM_GBS,
                            "traffic_bytes": counter_traffic(cfg_tag, args.layout, k1_inst, args.transform)}
        kernels[k2_name] = {"ms": k2_ms, "p10_ms": k2_p10, "p90_ms": k2_p90, "bound": "mfma", "ops": tap_ops,
                            "TOP/s": tap_ops / (k2_ms * 1e-3) / 1e12,
                            "frac": tap_ops / (k2_ms * 1e-3) / 1e12 / k2_peak,
                            "GB/s_algorithmic": k2_bytes / (k2_ms * 1e-3) / 1e9,
                            "traffic_bytes": counter_traffic(cfg_tag, args.layout, k2_inst, args.transform),
                            "stream_k": gemm == "rows_streamk"}
        # the input transform's HBM figures are taken cold (inputs in HBM,
        # caches flushed): warm, C5's 26 MB input sits in the 256 MB MALL
        k1c = cold["kernels_ms"][k1_name]
        kernels[k1_name].update({"warm_GB/s": kernels[k1_name]["GB/s"], "warm_frac": kernels[k1_name]["frac"],
                                 "cold_ms": k1c, "GB/s": k1_bytes / (k1c * 1e-3) / 1e9,
                                 "frac": k1_bytes / (k1c * 1e-3) / 1e9 / PEAK_HBM_GBS})
        kernels[k2_name]["cold_ms"] = cold["kernels_ms"][k2_name]
        if one_launch:
            # the step runs this kernel alone; K1 and K2 above are what
            # wino_f4_input_transform and wino_f4_tap_gemm would run
            two_launches, kernels = kernels, {cs_name: {
                "ms": cs_ms, "p10_ms": cs_p10, "p90_ms": cs_p90, "cold_ms": cold["step_ms"], "bound": "mfma",
                "ops": tap_ops, "TOP/s": tap_ops / (cs_ms * 1e-3) / 1e12,
                "frac": tap_ops / (cs_ms * 1e-3) / 1e12 / k2_peak,
                "GB/s_algorithmic": fused_min / (cs_ms * 1e-3) / 1e9,
                "traffic_bytes": counter_traffic(cfg_tag, args.layout, cs_inst, args.transform)}}
            roofline = {"kernel": cs_name, "bound": "mfma", "achieved": kernels[cs_name]["TOP/s"],
                        "peak": k2_peak, "unit": k2_unit, "frac": kernels[cs_name]["frac"],
                        "traffic": kernels[cs_name]["traffic_bytes"]}
        elif k2_ms >= k1_ms:
            roofline = {"kernel": k2_name, "bound": "mfma", "achieved": kernels[k2_name]["TOP/s"],
                        "peak": k2_peak, "unit": k2_unit, "frac": kernels[k2_name]["frac"],
                        "traffic": kernels[k2_name]["traffic_bytes"]}
        else:
            roofline = {"kernel": k1_name, "bound": "hbm", "achieved": kernels[k1_name]["GB/s"],
                        "peak": PEAK_HBM_GBS, "unit": "GB/s", "frac": kernels[k1_name]["frac"],
                        "traffic": kernels[k1_name]["traffic_bytes"]}
    else:
        roofline = {"kernel": "wino_fused", "bound": "mfma", "achieved": tap_ops / (ms * 1e-3) / 1e12,
                    "peak": PEAK_INT8_TOPS, "unit": "TOP/s",
                    "frac": tap_ops / (ms * 1e-3) / 1e12 / PEAK_INT8_TOPS, "traffic": None}

    # the chip's rates measured in this run: int8 MFMA loops (both shapes;
    # the tap GEMM issues 16x16x64) and a 1 GiB device copy (HBM-bound)
    measured = {}
    sink = torch.zeros(4, dtype=torch.int32, device="cuda")
    blocks = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    for shape in (32, 16):
        W.wino_probe_mfma_int8(shape, 100, blocks, sink)
        best = None
        for _ in range(3):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            s.record()
            ops_probe = W.wino_probe_mfma_int8(shape, 20000, blocks, sink)
            e.record()
            torch.cuda.synchronize()
            t = s.elapsed_time(e)
            best = t if best is None else min(best, t)
        name = "int8_mfma_32x32x32_TOPS" if shape == 32 else "int8_mfma_16x16x64_TOPS"
        measured[name] = ops_probe / (best * 1e-3) / 1e12
    src = torch.ones(1 << 30, dtype=torch.int8, device="cuda")
    dst = torch.empty_like(src)
    dst.copy_(src)
    best = None
    for _ in range(3):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        s.record()
        dst.copy_(src)
        e.record()
        torch.cuda.synchronize()
        best = s.elapsed_time(e) if best is None else min(best, s.elapsed_time(e))
    measured["hbm_copy_GBs"] = 2.0 * src.numel() / (best * 1e-3) / 1e9
    del src, dst
    if variant == W.SPLIT and args.bits == 8:
        split_kernels = two_launches or kernels
        split_kernels[k2_name]["frac_of_measured_32x32x32"] = (split_kernels[k2_name]["TOP/s"] /
                                                               measured["int8_mfma_32x32x32_TOPS"])
        split_kernels[k1_name]["frac_of_measured_copy"] = split_kernels[k1_name]["GB/s"] / measured["hbm_copy_GBs"]

    direct = None
    if not args.no_direct:
        wq, _ = W.direct_conv_quantize_weights(f)
        wd = torch.from_numpy(wq).cuda()
        bd = torch.from_numpy(np.asarray(bias, np.int32)).cuda()
        yd = torch.empty_like(y)

        def dstep():
            W.direct_conv_int8(xd, wd, bd, yd, n, cin, cout, h, w, layout, 8, spec.relu)

        for _ in range(max(2, args.warmup // 2)):
            dstep()
        dms, d10, d90 = kernel_ms(torch, dstep, max(5, args.steps // 2))
        direct = {"ms": dms, "p10_ms": d10, "p90_ms": d90, "TOPS": direct_ops / (dms * 1e-3) / 1e12, "speedup": dms / ms,
                  "mfma_frac": direct_ops / (dms * 1e-3) / 1e12 / PEAK_INT8_TOPS}

    cpu = None
    if not args.no_cpu_baseline:
        from oracle import tapwise
        oplan = tapwise.make_plan(f, eb, bias=bias, out_shift=out_shift, relu=spec.relu)
        cpu = cpu_baseline(x, oplan, args.cpu_images, spec, f)

    if args.copy_probe:
        src = torch.empty(256 << 20, dtype=torch.int8, device="cuda").fill_(1)
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)                    # runtime blit kernel
            torch.add(src, 0, out=dst)        # vectorized elementwise kernel, same bytes
        torch.cuda.synchronize()

    line = {
        "metric": METRIC, "value": value, "unit": "TOPS", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": ms, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "int8" if args.bits == 8 else "int8/int10", "data": "synthetic",
        "config": {"workload": f"{args.config}: {wl.desc}" + (f" (layer {args.layer})" if args.layer else "")
                   + (f", one GPU's share: {share}" if share else ""),
                   "n": n, "cin": cin, "cout": cout, "h": h, "w": w,
                   "layout": args.layout, "variant": args.variant, "transform": args.transform,
                   "winograd_bits": args.bits, "tiles": T,
                   "e_b": eb, "e_g": info["e_g"], "out_shift": out_shift,
                   "epilogue_bits": info["epilogue_bits"]},
        "roofline": roofline,
        "bitexact": bitexact,
        "kernels": kernels,
        "two_launches_not_in_step": two_launches,
        "tap_gemm_mfma_frac_of_step": tap_ops / (ms * 1e-3) / 1e12 / k2_peak,
        "layer_hbm": layer_hbm,
        "cold": {"step_ms": cold["step_ms"], "TOPS": direct_ops / (cold["step_ms"] * 1e-3) / 1e12,
                 "calls": ncold, "flush": "1 GiB read before each call (L2 and MALL evicted, clean)"},
        "measured_peaks": measured,
        "direct_conv": direct,
        "cpu_baseline": cpu,
        "plan_ms": plan_ms,
    }
    print(json.dumps(line), flush=True)
    if bitexact is False:
        sys.exit("bench: the timed output differs from the oracle's golden record")


if __name__ == "__main__":
    main()
