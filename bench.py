#!/usr/bin/env python3
"""Benchmark of the fused reduce + optimizer step on one MI355X.

A step is one fused reduce+Adam pass (chunk lookup, R-way fp16 reduce, unscale and overflow test, moments,
weight update, fp16 emission) over the BERT-Large parameter list with R = 8 gradient slices (configuration 2),
inputs resident in HBM.  The same run also times, with the same method, the four other configurations (the fused
LAMB step on that list, the GPT-2 1.5B list with Adam, the 1/8 shard of an 8.3B transformer with LAMB, and the
2^20-element tensor with eager launches, graph replay and evicted caches), the unfused reduce / optimizer / cast
pipelines, a plain copy kernel (the practical HBM ceiling) and the CPU oracle on a bounded sample.  One JSON line is
printed.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config 2] [--chunk-elems N] [--no-extras]
    python bench.py --mode sweep|rsweep|cold|sliced|epilogue|small   (measurement programs behind profiles/*.md, see bench_sweeps.py)
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published

# HBM bytes per launch of the headline kernel from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, each scaled by what
# the same counter reads for the plain copy kernel: default chunk size and schedule, fp16 slices, scattered list only.
# These are constants copied from the kept profiles, not measured by this run.
MEASURED_TRAFFIC = {2: (9.4217e9 + 4.7096e9, "profiles/fused_adam_config2.md"),
                    3: (1.3462e10 + 4.7132e9, "profiles/fused_lamb_config3.md"),
                    4: (4.3644e10 + 2.1818e10, "profiles/fused_adam_config4.md"),
                    5: (4.1621e10 + 1.4573e10, "profiles/fused_lamb_config5.md")}

WORKLOAD_NAMES = {1: "one flat tensor", 2: "BERT-Large parameter list", 3: "BERT-Large parameter list",
                  4: "GPT-2 1.5B parameter list", 5: "1/8 shard of an 8.3B transformer"}


def adam_bytes_per_param(R, gb=2):   # read gb R (gradient slices) + 12 (w, m, v); write 12 (w, m, v) + 2 (fp16 w)
    return gb * R + 26


def lamb_bytes_per_param(R, gb=2):   # phase 1: read gb R + 12, write 8; phase 2: read 12, write 6
    return gb * R + 38


def unfused_adam_bytes_per_param(R, gb=2):   # reduce: gb R + 4; optimizer: 16 + 12; cast: 4 + 2
    return gb * R + 38


def unfused_lamb_bytes_per_param(R, gb=2):   # reduce gb R + 4; phase 1: 16 + 8; phase 2: 12 + 4; cast 4 + 2
    return gb * R + 50


class Timer:
    """Times consecutive optimizer steps of one shard with HIP events on the launch stream (torch's current stream,
    which is also the stream the binding launches on)."""

    def __init__(self, torch, cc, shard, cfg, skip_mode=0):
        self.torch, self.cc, self.shard, self.cfg, self.skip_mode = torch, cc, shard, cfg, skip_mode
        self.t = 1

    def hyper(self, t):
        c = self.cfg
        return self.cc.Hyper(lr=c.lr, beta1=c.beta1, beta2=c.beta2, eps=c.eps, loss_scale=c.loss_scale, step=t,
                             skip_mode=self.skip_mode)

    def run(self, fn, steps, warmup, graph=False, per=100):
        """warmup + steps consecutive steps, each reading the copy the previous one wrote; events bracket exactly
        `steps` of them.  graph: the timed steps are replays of a captured graph of `per` steps (an even number, so that the
        ping-pong state is back where it started; the step count t is baked into the recording; every replay costs the
        device 4-5 us on top of its nodes, 0.2 us per step with 20 steps per graph and 0.05 us with 100).  Returns ms per step."""
        torch, shard = self.torch, self.shard
        for _ in range(warmup):
            shard.run(fn, self.hyper(self.t))
            shard.commit()
            self.t += 1
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        if graph:
            assert per % 2 == 0 and steps % per == 0, "graph replay needs an even number of steps per graph that divides the step count"
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                for i in range(per):
                    shard.run(fn, self.hyper(self.t + i))
                    shard.commit()
            for _ in range(max(1, warmup // per)):
                g.replay()
            torch.cuda.synchronize()
            e0.record()
            for _ in range(steps // per):
                g.replay()
            e1.record()
            torch.cuda.synchronize()
            self.t += per
        else:
            e0.record()
            for _ in range(steps):
                shard.run(fn, self.hyper(self.t))
                shard.commit()
                self.t += 1
            e1.record()
            torch.cuda.synchronize()
        assert int(shard.flag.item()) == 0, "overflow flag set during the timed run"
        return e0.elapsed_time(e1) / steps

    def cold(self, fn, evict, reps=30):
        """Median ms of one step whose caches were evicted first (evict() enqueues a copy far larger than the 256 MB
        Infinity Cache); the event pair brackets the step alone."""
        torch, shard = self.torch, self.shard
        times = []
        for _ in range(reps):
            evict()
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            shard.run(fn, self.hyper(self.t))
            b.record()
            shard.commit()
            self.t += 1
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        times.sort()
        return times[len(times) // 2]


# By the template argument of the first kernel.
POLICIES = (("12WriteThroughELb1E", "non-temporal loads but for the slices, write-through stores"), ("8Resident", "plain loads, write-through stores (cache-resident shard)"), ("12WriteThrough", "non-temporal loads, write-through stores"),
            ("11WeightsKept", "non-temporal loads but for the weights in the first sweep, write-through stores"))


def describe(cc, shard, R, optimizer, gf32):
    """What a step of this shard runs; the kernels are read from a captured graph of one step, which executes nothing."""
    from paper_2105_05720_amd.launches import launches
    chunk, block, _ = cc.cc_plan_layout(shard.plans[0])
    _, chunks, table_bytes = cc.cc_plan_info(shard.plans[0])
    fn = cc.cc_fused_adam_step if optimizer == "adam" else cc.cc_fused_lamb_step
    what = launches(lambda: shard.run(fn, cc.Hyper(step=1, skip_mode=int(shard.in_place))))
    kernel = " + ".join("%s<%s%d threads>" % (x.kernel, "R=%d, " % R if x.kernel.startswith(("fused_adam", "lamb_phase1", "lamb_one")) else "", x.block)
                        for x in what)
    if "_ordered_kernel" in what[0].kernel:
        schedule = "ordered: %d persistent workgroups take the chunks in table order" % what[0].grid
    elif what[0].grid != chunks and what[0].kernel.startswith("lamb"):
        schedule = "one workgroup of %d threads per chunk of 1024 elements" % what[0].block
    elif what[0].grid != chunks:
        schedule = "%d workgroups of %d threads, one per piece of 256 elements" % (what[0].grid, what[0].block)
    else:
        schedule = "one workgroup of %d threads per chunk" % what[0].block
    return {"chunk_elems": chunk, "chunks": chunks, "table_bytes": table_bytes, "kernel": kernel, "schedule": schedule,
            "cache_policy": next((text for name, text in POLICIES if name in what[0].symbol), "non-temporal accesses")}


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--mode", choices=("step", "sweep", "rsweep", "cold", "sliced", "epilogue", "small"), default="step",
                    help="step: the benchmark line (default); the others are the measurement programs of bench_sweeps.py")
    ap.add_argument("--config", type=int, default=2, help="workload configuration 1..5 (default 2, the metric's)")
    ap.add_argument("--chunk-elems", type=int, default=0)
    ap.add_argument("--in-place", action="store_true", help="in-place state with the per-element guard (skip_mode 1)")
    ap.add_argument("--grad-dtype", choices=("f16", "f32"), default="f16", help="element type of the R gradient slices")
    ap.add_argument("--flat", action="store_true", help="the same number of parameters as ONE contiguous tensor (Table 2's single-tensor case)")
    ap.add_argument("--graph", action="store_true", help="enqueue the timed steps as replays of a captured HIP graph of --graph-steps steps")
    ap.add_argument("--graph-steps", type=int, default=100, help="steps per captured graph (even)")
    ap.add_argument("--schedule", choices=("auto", "per-chunk", "ordered", "tuned"), default="auto",
                    help="how the kernels are laid over the device (cc_plan_set_schedule); auto = the library's size rule, "
                         "tuned = cc_plan_autotune measures the candidates on this workload first")
    ap.add_argument("--cache", choices=("auto", "streaming", "resident", "write-through"), default="auto", help="cc_plan_set_cache_policy")
    ap.add_argument("--workgroups", type=int, default=0, help="workgroups of the ordered schedule (0 = one per compute unit)")
    ap.add_argument("--no-extras", action="store_true", help="only the headline step (for profiling runs)")
    ap.add_argument("--copy-only", action="store_true", help="run only the plain copy kernel (2 GiB, 20 launches): counter calibration")
    ap.add_argument("--cpu-seconds", type=float, default=15.0, help="target CPU time of the oracle sample")
    args, rest = ap.parse_known_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build measures one GPU's shard only (no collectives, no sharding across GPUs); "
              "run it with --gpus 1", file=sys.stderr)
        return 2

    import torch

    from paper_2105_05720_amd import binding as cc
    from paper_2105_05720_amd import workloads as W
    from paper_2105_05720_amd.shard import Shard

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    cc.load()                                            # raises if libccfused.so is missing
    torch.cuda.set_device(0)
    dev = torch.device("cuda:0")
    if args.mode != "step":
        import bench_sweeps
        return bench_sweeps.main(args.mode, rest)
    if rest:
        ap.error("unknown arguments: %s" % " ".join(rest))
    if args.copy_only:
        nbytes = 2 << 30
        src = torch.empty(nbytes, dtype=torch.uint8, device=dev).fill_(1)
        dst = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        for _ in range(20):
            cc.cc_copy_probe(dst, src, nbytes)
        torch.cuda.synchronize()
        print(json.dumps({"copy_only": True, "bytes_read_per_launch": nbytes, "bytes_written_per_launch": nbytes, "launches": 20}))
        return 0

    gb = 2 if args.grad_dtype == "f16" else 4
    K, Wm = args.steps, args.warmup
    sched_arg = {"auto": cc.CC_SCHEDULE_AUTO, "per-chunk": cc.CC_SCHEDULE_PER_CHUNK, "ordered": cc.CC_SCHEDULE_ORDERED,
                 "tuned": cc.CC_SCHEDULE_AUTO}[args.schedule]
    cache_arg = {"auto": cc.CC_CACHE_AUTO, "streaming": cc.CC_CACHE_STREAMING, "resident": cc.CC_CACHE_RESIDENT,
                 "write-through": cc.CC_CACHE_WRITE_THROUGH}[args.cache]
    default_options = (args.chunk_elems == 0 and not args.in_place and not args.flat and args.grad_dtype == "f16"
                       and args.schedule == "auto" and args.workgroups == 0 and args.cache == "auto")

    def make(index, options=True, unfused=False):
        """(config, shard with state and the first call's gradients in HBM)"""
        cfg = W.config(index)
        if options and args.flat:
            import dataclasses
            cfg = dataclasses.replace(cfg, params=(W.ParamSpec("flat", cfg.numel, "matrix"),))
        kw = dict(chunk_elems=args.chunk_elems, in_place=args.in_place, schedule=sched_arg, workgroups=args.workgroups,
                  cache_policy=cache_arg,
                  grad_dtype=torch.float16 if args.grad_dtype == "f16" else torch.float32) if options else {}
        shard = Shard([s.numel for s in cfg.params], [cfg.wd_of(s) for s in cfg.params], cfg.R, device=dev, unfused=unfused, **kw)
        W.fill_state(shard, cfg)
        W.fill_grads(shard, cfg, 1)
        torch.cuda.synchronize()
        return cfg, shard

    def rate(ms, bytes_pp, N):
        gbs = bytes_pp * N / (ms * 1e-3) / 1e9
        return {"ms_per_step": round(ms, 5), "GB/s": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4),
                "params_per_sec": round(N / (ms * 1e-3), 1), "algorithmic_bytes_per_param": bytes_pp}

    cfg, shard = make(args.config, unfused=not args.no_extras)
    R, N = cfg.R, cfg.numel
    tuned = None
    if args.schedule == "tuned":
        assert not args.in_place, "--schedule tuned needs out-of-place state"
        hp1 = cc.Hyper(lr=cfg.lr, beta1=cfg.beta1, beta2=cfg.beta2, eps=cfg.eps, loss_scale=cfg.loss_scale, step=1)
        tuned = [cc.cc_plan_autotune(p, hp1, shard.flag, 0 if cfg.optimizer == "adam" else 1) for p in shard.plans]
    timer = Timer(torch, cc, shard, cfg, skip_mode=1 if args.in_place else 0)
    headline_fn = cc.cc_fused_adam_step if cfg.optimizer == "adam" else cc.cc_fused_lamb_step
    bpp = adam_bytes_per_param(R, gb) if cfg.optimizer == "adam" else lamb_bytes_per_param(R, gb)

    # ---- the K timed steps of the headline path -------------------------------------------------------------
    torch.cuda.synchronize()
    wall0 = time.perf_counter()
    ms = timer.run(headline_fn, K, Wm, graph=args.graph, per=args.graph_steps)
    wall = time.perf_counter() - wall0
    gbs = bpp * N / (ms * 1e-3) / 1e9
    what = describe(cc, shard, R, cfg.optimizer, gb == 4)
    traffic = MEASURED_TRAFFIC.get(cfg.index) if default_options else None
    out = {
        "metric": "fused reduce+optimizer HBM GB/s (% of MI355X peak) and params updated/sec",
        "value": round(gbs, 1), "unit": "GB/s",
        "pct_of_peak": round(100 * gbs / HBM_PEAK_GBS, 2),
        "params_per_sec": round(N / (ms * 1e-3), 1),
        "n_gpus": 1, "steps": K, "warmup": Wm, "ms_per_step": round(ms, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32", "data": "synthetic",
        "config": {"workload": "config %d: fused %s, %s, T=%d tensors, N=%d fp32 params, R=%d fp16 gradient slices, "
                               "%s state" % (cfg.index, cfg.optimizer,
                                             "the same N as ONE contiguous tensor" if args.flat else WORKLOAD_NAMES[cfg.index],
                                             len(cfg.params), N, R, "in-place" if args.in_place else "out-of-place (ping-pong)") + (
                                                 " [fp32 gradient slices]" if args.grad_dtype == "f32" else ""),
                   "chunk_elems": what["chunk_elems"], "chunks": what["chunks"],
                   "launch": "hip graph replay" if args.graph else "eager",
                   "schedule": what["schedule"], "cache_policy": what["cache_policy"],
                   "autotune_ms_best_and_per_chunk": [round(x, 5) for x in tuned[0]] if tuned else None,
                   "table_bytes": what["table_bytes"], "algorithmic_bytes_per_param": bpp},
        "roofline": {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": round(gbs / HBM_PEAK_GBS, 4),
                     "traffic": traffic[0] if traffic else None,
                     "traffic_source": ("constant from %s (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, scaled by the copy kernel); "
                                        "not measured by this run" % traffic[1]) if traffic else None,
                     "kernel": what["kernel"], "bytes_per_launch": bpp * N, "avg_launch_ms": round(ms, 5)},
    }

    if not args.no_extras:
        extras = {}
        t_next = timer.t
        # the same K steps with the flag read back (and the commit decided) after every step
        for _ in range(3):
            shard.step(headline_fn, timer.hyper(t_next)); t_next += 1
        torch.cuda.synchronize()
        w0 = time.perf_counter()
        for _ in range(K):
            assert shard.step(headline_fn, timer.hyper(t_next)) == 0
            t_next += 1
        extras["ms_per_step_with_flag_readback"] = round((time.perf_counter() - w0) * 1e3 / K, 5)
        extras["wall_ms_per_step_enqueue_only_loop"] = round(wall * 1e3 / (K + Wm), 5)
        timer.t = t_next

        ks = max(5, K // 4)
        if args.graph:
            ks = max(20, ks // 20 * 20)
        wk = max(2, Wm // 2)
        if cfg.optimizer == "adam":
            extras["fused_lamb_same_list"] = rate(timer.run(cc.cc_fused_lamb_step, ks, wk, args.graph), lamb_bytes_per_param(R, gb), N) if not args.in_place else None
        else:
            extras["fused_adam_same_list"] = rate(timer.run(cc.cc_fused_adam_step, ks, wk, args.graph), adam_bytes_per_param(R, gb), N)
        extras["unfused_adam"] = rate(timer.run(cc.cc_unfused_adam_step, ks, wk, args.graph), unfused_adam_bytes_per_param(R, gb), N)
        if args.grad_dtype == "f16":          # reduce 2R + 2, optimizer 14 + 12, cast 4 + 2
            extras["unfused_adam_fp16_intermediate"] = rate(timer.run(
                lambda p, h, f, st=None: cc.cc_unfused_adam_step_ex(p, h, f, st, cc.CC_GRAD_F16), ks, wk, args.graph), 2 * R + 34, N)
        if not args.in_place:
            extras["unfused_lamb"] = rate(timer.run(cc.cc_unfused_lamb_step, ks, wk, args.graph), unfused_lamb_bytes_per_param(R, gb), N)
        fa = extras.get("fused_adam_same_list", {"ms_per_step": ms})["ms_per_step"] if cfg.optimizer != "adam" else ms
        extras["fused_vs_unfused_adam_speedup"] = round(extras["unfused_adam"]["ms_per_step"] / fa, 3)

        out["cpu_baseline"] = cpu_baseline(shard, cfg, timer.hyper(1), args.cpu_seconds)
        shard.destroy()
        del shard, timer
        torch.cuda.empty_cache()

        # plain copy kernel: the practical streaming ceiling of this machine (bytes counted once read + once written)
        nbytes = 2 << 30
        src = torch.empty(nbytes, dtype=torch.uint8, device=dev).fill_(1)
        dst = torch.empty(nbytes, dtype=torch.uint8, device=dev)
        for _ in range(3):
            cc.cc_copy_probe(dst, src, nbytes)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            cc.cc_copy_probe(dst, src, nbytes)
        e1.record()
        torch.cuda.synchronize()
        extras["copy_kernel_GB/s"] = round(2 * nbytes / (e0.elapsed_time(e1) / 20 * 1e-3) / 1e9, 1)

        # ---- the other configurations, default options, same timing method ---------------------------------------
        if default_options and not args.graph:
            others = {}
            for index in (1, 3, 4, 5):
                if index == cfg.index:
                    continue
                c2, s2 = make(index, options=False)
                t2 = Timer(torch, cc, s2, c2)
                fn2 = cc.cc_fused_adam_step if c2.optimizer == "adam" else cc.cc_fused_lamb_step
                b2 = adam_bytes_per_param(c2.R) if c2.optimizer == "adam" else lamb_bytes_per_param(c2.R)
                rec = {"workload": "config %d: fused %s, %s, T=%d, N=%d, R=%d" % (index, c2.optimizer, WORKLOAD_NAMES[index],
                                                                                  len(c2.params), c2.numel, c2.R)}
                rec.update(describe(cc, s2, c2.R, c2.optimizer, False))
                if b2 * c2.numel < (256 << 20):
                    # the whole step fits the 256 MB Infinity Cache: consecutive steps run cache-resident, and an eager
                    # launch loop measures the Python caller; so all four combinations are reported
                    rec["warm_cache_hip_graph_replay"] = rate(t2.run(fn2, 4000, 400, graph=True), b2, c2.numel)
                    rec["warm_cache_eager_launches"] = rate(t2.run(fn2, 2000, 200), b2, c2.numel)
                    rec["cold_cache_single_step"] = rate(t2.cold(fn2, lambda: cc.cc_copy_probe(dst, src, nbytes)), b2, c2.numel)
                    rec["note"] = ("cache-resident: GB/s here is not HBM bandwidth; cold = caches evicted by a 2 GiB copy before "
                                   "every step, the event pair brackets the step alone (launch mode does not enter)")
                    rec.update(rec["warm_cache_hip_graph_replay"])
                    rec["launch"] = "hip graph replay"
                else:
                    n2 = max(10, min(K, int(400.0 / (b2 * c2.numel / 6.4e12 * 1e3))))   # about 0.4 s of steps
                    rec.update(rate(t2.run(fn2, n2, max(3, n2 // 8)), b2, c2.numel))
                    rec["launch"] = "eager"
                    rec["steps"] = n2
                tr = MEASURED_TRAFFIC.get(index)
                rec["traffic"] = tr[0] if tr else None
                rec["traffic_source"] = ("constant from %s; not measured by this run" % tr[1]) if tr else None
                others["config%d" % index] = rec
                s2.destroy()
                del s2, t2
                torch.cuda.empty_cache()
            extras["configs"] = others
        del src, dst
        cus, clk_khz, bus_bits, total_bytes = cc.cc_device_info()
        extras["device"] = {"name": torch.cuda.get_device_name(0), "compute_units": cus, "memory_clock_khz": clk_khz,
                            "memory_bus_bits": bus_bits, "total_GiB": round(total_bytes / 2 ** 30, 1),
                            # HBM3E moves 4 bits per pin per reported (command) clock: 2 GHz -> 8 Gb/s per pin;
                            # 8192 pins x 8 Gb/s / 8 = 8192 GB/s, the published 8 TB/s
                            "GB/s_at_4_transfers_per_clock": round(4 * clk_khz * 1e3 * bus_bits / 8 / 1e9, 1)}
        out["extras"] = extras
    else:
        shard.destroy()

    print(json.dumps(out), flush=True)
    return 0


def cpu_baseline(shard, cfg, ghp, target_seconds):
    """The CPU oracle, as it stands, on a bounded sample of the same workload: the first tensors of the list up to
    a parameter budget sized from a short calibration run, all host threads (whole tensors per thread)."""
    import numpy as np

    import oracle

    threads = min(16, len(os.sched_getaffinity(0)))
    step_fn = oracle.adam_step if cfg.optimizer == "adam" else oracle.lamb_step
    ohp = oracle.Hyper(lr=ghp.lr, beta1=ghp.beta1, beta2=ghp.beta2, eps=ghp.eps, loss_scale=ghp.loss_scale, step=1)
    bits = lambda t: t.cpu().view(__import__("torch").int16).numpy().view(np.uint16).copy()

    def tensors_of(ks):
        return [oracle.OracleTensor(w=shard.w_of(k).cpu().numpy().copy(), m=shard.m_of(k).cpu().numpy().copy(),
                                    v=shard.v_of(k).cpu().numpy().copy(),
                                    grads=[bits(shard.grad_of(r, k)) for r in range(cfg.R)],
                                    weight_decay=shard.wds[k]) for k in ks]

    # calibrate on a few small tensors, then take tensors in list order (the giant embeddings last, they keep
    # one thread busy on their own) until the time budget is filled or the list ends
    small = [k for k, s in enumerate(cfg.params) if 0 < s.numel <= 8_000_000]
    order = small + [k for k, s in enumerate(cfg.params) if s.numel > 8_000_000]
    calib = []
    budget = 2_000_000
    for k in order:
        calib.append(k)
        budget -= cfg.params[k].numel
        if budget <= 0:
            break
    ots = tensors_of(calib)
    t0 = time.perf_counter()
    step_fn(ots, ohp, threads=threads)
    rate = sum(cfg.params[k].numel for k in calib) / (time.perf_counter() - t0)
    want = rate * target_seconds
    sample, total = [], 0
    for k in order:
        if total >= want:
            break
        sample.append(k)
        total += cfg.params[k].numel
    ots = tensors_of(sample)
    t0 = time.perf_counter()
    step_fn(ots, ohp, threads=threads)
    dt = time.perf_counter() - t0
    # the definition itself: one thread, on the calibration tensors
    ots1 = tensors_of(calib)
    t0 = time.perf_counter()
    step_fn(ots1, ohp, threads=1)
    single = sum(cfg.params[k].numel for k in calib) / (time.perf_counter() - t0)
    bpp = adam_bytes_per_param(cfg.R) if cfg.optimizer == "adam" else lamb_bytes_per_param(cfg.R)
    return {"single_thread_params_per_sec": round(single, 1),
            "value": round(bpp * total / dt / 1e9, 4), "unit": "GB/s", "params_per_sec": round(total / dt, 1),
            "cores": threads, "kind": "oracle", "seconds": round(dt, 2),
            "sample": "%d of the %d tensors of the same list (%d params), one %s step, whole tensors spread over %d threads" % (
                len(sample), len(cfg.params), total, cfg.optimizer, threads)}


if __name__ == "__main__":
    sys.exit(main())
