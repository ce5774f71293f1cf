#!/usr/bin/env python3
"""Benchmark of the dedup dispatch + combine hot path on one MI355X.

A step is one pass of the whole forward path over one batch of synthetic routing and
activations already resident in HBM:
    hm_plan (+ the expert-load counts) -> hm_dispatch_pack -> (identity experts) -> hm_combine
Headline workload: the DeepSeek-V3-shaped layer (T=8192, H=7168, E=256, top-8 group-limited,
4 nodes x 8 ranks, node-level dedup).  The default run then times every other workload / dedup
level of the benchmark set the same way and adds them as the `configs` table of the ONE JSON line
it prints on stdout; details go to stderr.

  python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload dsv3] [--level node] [--no-table]
"""
from __future__ import annotations

import argparse
import ctypes
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published peak
LEVELS = {"none": 0, "gpu": 1, "node": 2}
# every other configuration of the benchmark set, timed after the headline one
TABLE = [("tiny", "none"), ("tiny", "gpu"), ("tiny", "node"), ("qwen3", "gpu"), ("qwen3", "node"),
         ("dsv3", "gpu"), ("dsv3", "none"), ("skew", "gpu"), ("skew", "node"), ("skew-swapped", "gpu"),
         ("skew-swapped", "node"), ("stress", "node"), ("stress", "gpu")]


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def rows_source_digest() -> str:
    """Identifies the row kernels a counter summary was taken on: the first 16 hex digits of the
    SHA-256 of their source file."""
    path = os.path.join(ROOT, "paper_2508_09591_amd", "csrc", "hm_rows.hip")
    return hashlib.sha256(open(path, "rb").read()).hexdigest()[:16]


def measured_traffic(workload: str, level: str, kernel: str):
    """HBM bytes per launch from the committed rocprofv3 counter summaries: lines
    `traffic <workload> <level> <entry point> <bytes> <digest of hm_rows.hip>` under profiles/.
    A figure taken on other kernel sources than the ones in the tree is not used (None)."""
    pdir = os.path.join(ROOT, "profiles")
    if not os.path.isdir(pdir):
        return None
    digest = rows_source_digest()
    for name in sorted(os.listdir(pdir)):
        if not name.endswith(".txt"):
            continue
        for line in open(os.path.join(pdir, name)):
            f = line.split()
            if len(f) == 6 and f[0] == "traffic" and f[1:4] == [workload, level, kernel] and f[5] == digest:
                return int(f[4])
    return None


_probe = None


def stream_probe(src, read_streams, dst, write_streams, block_threads=64, waves_per_cu=32, stream=None):
    """Flat-stream reference kernel of libhmprobe.so (built beside the library, used by this
    benchmark only): dst[j] = XOR_i src[i] over 16-byte vectors, with the given launch shape."""
    global _probe
    import torch
    if _probe is None:
        path = os.path.join(ROOT, "paper_2508_09591_amd", "libhmprobe.so")
        if not os.path.exists(path):
            raise RuntimeError("libhmprobe.so is not built (run __graft_entry__.build())")
        _probe = ctypes.CDLL(path)
        _probe.bench_stream_probe.restype = ctypes.c_int
        _probe.bench_stream_probe.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int32,
                                              ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
    if not (src.is_cuda and dst.is_cuda and src.is_contiguous() and dst.is_contiguous()):
        raise TypeError("src and dst must be contiguous GPU tensors")
    nbytes = src.numel() * src.element_size()
    n = nbytes // (16 * read_streams)
    if nbytes != n * 16 * read_streams or dst.numel() * dst.element_size() != n * 16 * write_streams:
        raise ValueError("src / dst sizes do not match the stream counts")
    s = torch.cuda.current_stream() if stream is None else stream
    rc = _probe.bench_stream_probe(src.data_ptr(), read_streams, dst.data_ptr(), write_streams, n, block_threads,
                                   waves_per_cu, s.cuda_stream or None)
    if rc != 0:
        raise RuntimeError("bench_stream_probe failed: %d" % rc)
    return dst


_event_overhead = {}


def event_pair_overhead_ms(stream):
    """What a start / stop pair of HIP events reads with nothing between them (median of 200 pairs
    on `stream`): the markers' own cost, which every per-call figure below would otherwise carry.
    It is measured once per stream and reported beside the per-call times (not subtracted: with a
    kernel between the markers part of it hides behind the kernel)."""
    import torch
    key = stream.cuda_stream
    if key not in _event_overhead:
        pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(200)]
        for a, b in pairs:
            a.record(stream)
            b.record(stream)
        torch.cuda.synchronize()
        _event_overhead[key] = sorted(a.elapsed_time(b) for a, b in pairs)[100]
    return _event_overhead[key]


def get_workload(name):
    """A workload of the benchmark set plus the placement to use: `skew-swapped` is the skew layer
    under its seeded random expert placement."""
    from paper_2508_09591_amd import workloads as W
    if name == "skew-swapped":
        return W.WORKLOADS["skew"], "expert_to_rank_swapped"
    return W.WORKLOADS[name], None


def time_send(wl, level, steps, warmup, nsets, *, label=None, placement_key=None, host_x=True, fused=True,
              explicit_weights=False, warm_y=False, graph=False, warm_leg=False, transposes=False, with_f32=False):
    """Times `steps` steps of the send path on one workload / level.  Returns a dict with the step
    time, the per-call HIP-event times, algorithmic bytes and rates, and what is needed for a CPU
    baseline (`routing`, `x_host`)."""
    import numpy as np
    import torch
    from paper_2508_09591_amd import binding as B
    from paper_2508_09591_amd import workloads as W

    level_name = W.LEVEL_NAMES[level]
    label = label or wl.name
    T, K, H, E = wl.T, wl.K, wl.H, wl.E
    t0 = time.time()
    r = W.make_routing(wl)
    e2r = r.extras[placement_key] if placement_key else r.expert_to_rank
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ids_d, w_d, e2r_d = dev(r.topk_ids), dev(r.topk_weights), dev(e2r)
    x = None
    if host_x:      # the seeded activations of the workload (what the CPU baseline also uses)
        x = W.make_activations(wl)
        x0 = dev(x.view(np.int16)).view(torch.bfloat16)
    else:           # same distribution, drawn on the GPU: the table rows do not feed a CPU run
        gen = torch.Generator(device="cuda")
        gen.manual_seed(1234 + wl.seed)
        x0 = torch.randn((T, H), dtype=torch.float32, device="cuda", generator=gen).to(torch.bfloat16)
    log("%s level %s: inputs ready in %.1f s" % (label, level_name, time.time() - t0))

    stream = torch.cuda.Stream()          # default priority
    cw_d = w_d if explicit_weights else None      # None: hm_combine takes the weights hm_plan merged
    plan = B.alloc_plan(T, K, E, wl.nodes, wl.ranks_per_node, level, loads=fused)
    with torch.cuda.stream(stream):
        B.hm_plan(ids_d, w_d, e2r_d, wl.nodes, wl.ranks_per_node, level, plan=plan)
        st, total_rows = B.hm_plan_status(plan)
    assert st == 0, B.status_string(st)
    c = total_rows / T
    nsets = max(1, nsets)
    xs = [x0] + [x0.clone() for _ in range(nsets - 1)]
    packs = [torch.empty((total_rows, H), dtype=torch.bfloat16, device="cuda") for _ in range(nsets)]
    outs = [torch.empty((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(nsets)]
    le = torch.empty(E, dtype=torch.int32, device="cuda")
    lr = torch.empty(wl.G, dtype=torch.int32, device="cuda")
    ln = torch.empty(wl.nodes, dtype=torch.int32, device="cuda")
    log("workload %s level %s: T=%d H=%d K=%d E=%d %dx%d ranks, rows=%d (c=%.3f), %d buffer sets = %.2f GB"
        % (label, level_name, T, H, K, E, wl.nodes, wl.ranks_per_node, total_rows, c, nsets,
           nsets * (2 * T + total_rows) * H * 2 / 1e9))

    # Expert outputs arrive from the exchange, not from this GPU's caches: combine therefore reads
    # the pack buffer written sets/2 steps earlier.  With identity experts and identical X copies
    # it holds the same rows as the one dispatch has just written.
    y_shift = 0 if warm_y else nsets // 2
    with torch.cuda.stream(stream):
        for s in range(nsets):
            B.hm_dispatch_pack(xs[s], plan, packs[s], stream=stream)
    torch.cuda.synchronize()

    def step(i, ev=None):
        # ev: a start and a stop event per call, each pair recorded around its own call only, so that
        # the marker between two calls is charged to neither
        s = i % nsets
        ys = (s + y_shift) % nsets
        if ev: ev[0].record(stream)
        B.hm_plan(ids_d, w_d, e2r_d, wl.nodes, wl.ranks_per_node, level, plan=plan, stream=stream)
        if ev: ev[1].record(stream); ev[2].record(stream)
        if not fused:        # otherwise hm_plan has already produced the three load arrays
            B.hm_expert_load(ids_d, e2r_d, wl.nodes, wl.ranks_per_node, le, lr, ln, stream=stream)
        if ev: ev[3].record(stream); ev[4].record(stream)
        B.hm_dispatch_pack(xs[s], plan, packs[s], stream=stream)
        if ev: ev[5].record(stream); ev[6].record(stream)
        B.hm_combine(packs[ys], cw_d, plan, outs[s], stream=stream)     # identity experts: Y = packed rows
        if ev: ev[7].record(stream)

    # ---- warm-up, then the timed region: exactly `steps` steps between two synchronisations ----
    run = step
    if graph:
        # The entry points only enqueue kernels, so a step records into a HIP graph as it is.
        for i in range(nsets):
            step(i)
        torch.cuda.synchronize()
        graphs = []
        for i in range(nsets):
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                step(i)
            graphs.append(g)
        run = lambda i: graphs[i % nsets].replay()
    for i in range(warmup):
        run(i)
    torch.cuda.synchronize()
    t_begin = time.perf_counter()
    for i in range(steps):
        run(i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t_begin
    ms_per_step = elapsed * 1e3 / steps

    # ---- per-kernel durations: the same steps again with HIP events on the launch stream ------
    events = [[torch.cuda.Event(enable_timing=True) for _ in range(8)] for _ in range(steps)]
    for i in range(steps):
        step(i, events[i])
    torch.cuda.synchronize()
    names = ["hm_plan", "hm_expert_load", "hm_dispatch_pack", "hm_combine"]
    ov = event_pair_overhead_ms(stream)
    per_call = {n: sorted(e[2 * j].elapsed_time(e[2 * j + 1]) for e in events) for j, n in enumerate(names)}
    avg_ms = {n: sum(v) / len(v) for n, v in per_call.items()}
    # An empty event pair already reads `ov`; with a kernel between the markers part of that cost hides
    # behind the kernel, so the kernel's own duration lies between (reading - ov) and the reading.  The
    # reading -- the conservative end -- is what every rate and roofline fraction below uses.
    low_avg_ms = {n: max(avg_ms[n] - ov, 0.0) for n in names}
    min_ms = {n: v[0] for n, v in per_call.items()}
    med_ms = {n: v[len(v) // 2] for n, v in per_call.items()}

    # the same two kernels back to back on ONE buffer set (inputs may sit in the 256 MB Infinity
    # Cache): reported beside the cold figures, never used for `value` or the roofline fraction
    warm_ms = {"hm_dispatch_pack": None, "hm_combine": None}
    if warm_leg:
        wev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(steps)]
        for e in wev:
            e[0].record(stream)
            B.hm_dispatch_pack(xs[0], plan, packs[0], stream=stream)
            e[1].record(stream)
            B.hm_combine(packs[0], cw_d, plan, outs[0], stream=stream)
            e[2].record(stream)
        torch.cuda.synchronize()
        warm_ms = {"hm_dispatch_pack": sorted(e[0].elapsed_time(e[1]) for e in wev)[len(wev) // 2],
                   "hm_combine": sorted(e[1].elapsed_time(e[2]) for e in wev)[len(wev) // 2]}     # one marker between the two calls: not corrected

    # correctness of what was timed: identity experts + weights summing to 1 -> output == input
    assert torch.equal(outs[(steps - 1) % nsets], xs[(steps - 1) % nsets]), "round trip failed"
    st, tr = B.hm_plan_status(plan, stream=stream)
    assert st == 0 and tr == total_rows
    loads = (plan.load_expert, plan.load_rank, plan.load_node) if fused else (le, lr, ln)
    assert int(loads[0].sum().item()) == T * K and int(loads[2].sum().item()) >= T

    row_bytes = 2 * H
    alg_bytes = {"hm_dispatch_pack": (1 + c) * T * row_bytes, "hm_combine": (c + 1) * T * row_bytes}
    kern = {}
    for n in ("hm_dispatch_pack", "hm_combine"):
        gbs = alg_bytes[n] / (avg_ms[n] * 1e-3) / 1e9
        kern[n] = {"avg_ms": round(avg_ms[n], 5), "median_ms": round(med_ms[n], 5), "min_ms": round(min_ms[n], 5),
                   "avg_ms_less_empty_event_pair": round(low_avg_ms[n], 5),
                   "warm_single_set_median_ms": None if warm_ms[n] is None else round(warm_ms[n], 5), "alg_bytes": int(alg_bytes[n]),
                   "achieved_GBps": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4),
                   "traffic": measured_traffic(label, level_name, n)}
        if kern[n]["traffic"]:      # HBM bytes the counters saw per launch over this run's launch time
            kern[n]["counter_GBps"] = round(kern[n]["traffic"] / (avg_ms[n] * 1e-3) / 1e9, 1)
            kern[n]["traffic_over_algorithmic"] = round(kern[n]["traffic"] / alg_bytes[n], 4)
    pair_ms = avg_ms["hm_dispatch_pack"] + avg_ms["hm_combine"]
    pair_gbs = (alg_bytes["hm_dispatch_pack"] + alg_bytes["hm_combine"]) / (pair_ms * 1e-3) / 1e9
    log("per-call (HIP events, avg/median/min ms; an empty event pair reads %.1f us): " % (ov * 1e3)
        + ", ".join("%s %.4f/%.4f/%.4f" % (n, avg_ms[n], med_ms[n], min_ms[n]) for n in names))
    if warm_leg:
        log("warm, one buffer set (median ms): dispatch %.4f, combine %.4f" % (warm_ms["hm_dispatch_pack"], warm_ms["hm_combine"]))
    log("dispatch+combine: %.4f ms -> %.1f GB/s algorithmic = %.1f%% of %.0f GB/s; %.2f M tokens/s (pair only); step %.4f ms"
        % (pair_ms, pair_gbs, 100 * pair_gbs / HBM_PEAK_GBS, HBM_PEAK_GBS, T / (pair_ms * 1e-3) / 1e6, ms_per_step))

    def timed(fn, nbytes, what):
        evs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
        with torch.cuda.stream(stream):
            for i in range(max(2, warmup)):
                fn()
            for a, b in evs:
                a.record(stream)
                fn()
                b.record(stream)
        torch.cuda.synchronize()
        tms = sum(a.elapsed_time(b) for a, b in evs) / len(evs)
        gbs = nbytes / (tms * 1e-3) / 1e9
        log("%s: %.4f ms -> %.1f GB/s algorithmic (%.1f%% of peak)" % (what, tms, gbs, 100 * gbs / HBM_PEAK_GBS))
        return {"avg_ms": round(tms, 5), "alg_bytes": int(nbytes), "achieved_GBps": round(gbs, 1),
                "frac": round(gbs / HBM_PEAK_GBS, 4)}

    extra = {}
    if transposes:      # the backward row of the 64 Ki-token layer: gradients back to the packed layout
        gout = torch.randn((T, H), dtype=torch.float32, device="cuda") * 1e-2
        gy = torch.empty((total_rows, H), dtype=torch.float32, device="cuda")
        tb = (1 + c) * T * 4 * H
        extra["hm_combine_transpose"] = timed(lambda: B.hm_combine_transpose(gout, plan, gy, stream=stream), tb,
                                              "hm_combine_transpose")
        del gy
        gout16 = gout.to(torch.bfloat16)
        gy16 = torch.empty((total_rows, H), dtype=torch.bfloat16, device="cuda")
        extra["hm_combine_transpose_bf16"] = timed(lambda: B.hm_combine_transpose_bf16(gout16, plan, gy16, stream=stream),
                                                   tb / 2, "hm_combine_transpose_bf16")
        del gout, gout16, gy16
    if with_f32:
        y32 = torch.randn((total_rows, H), dtype=torch.float32, device="cuda")
        o32 = torch.empty((T, H), dtype=torch.float32, device="cuda")
        extra["hm_combine_f32"] = timed(lambda: B.hm_combine_f32(y32, cw_d, plan, o32, stream=stream),
                                        (1 + c) * T * 4 * H, "hm_combine_f32")
        del y32, o32

    res = {"label": label, "level": level_name, "T": T, "H": H, "K": K, "E": E, "nodes": wl.nodes, "rpn": wl.ranks_per_node,
           "total_rows": total_rows, "c": c, "nsets": nsets, "y_shift": y_shift, "ms_per_step": ms_per_step,
           "tokens_per_s": T / (elapsed / steps), "kern": kern, "pair_ms": pair_ms, "pair_gbs": pair_gbs,
           "plan_ms": avg_ms["hm_plan"], "expert_load_ms": None if fused else avg_ms["hm_expert_load"], "event_overhead_ms": ov,
           "alg_bytes": alg_bytes, "extra": extra, "routing": r, "e2r": e2r, "x_host": x, "stream": stream}
    del xs, packs, outs
    torch.cuda.empty_cache()
    return res


def flat_stream_references(c, total_bytes, nsets, stream):
    """Context for the roofline fractions: flat streams with the read : write mix of the two row
    kernels and NO indirection, at the same total bytes.  For every mix the probe kernel's launch
    shape (workgroup size, cap on resident waves per CU) is swept and the best median is kept."""
    import torch
    cr = max(1, min(16, int(round(c))))
    mixes = [(1, 1), (1, cr), (cr, 1)] if cr > 1 else [(1, 1)]    # a plain copy, dispatch's mix, combine's mix
    shapes = [(b, w) for b in (64, 256) for w in (32, 24, 20, 16, 12, 8)]
    total_vec = int(total_bytes) // 16
    out = {}
    for nr, nw in mixes:
        n = total_vec // (nr + nw)
        srcs = [torch.empty((nr, n, 4), dtype=torch.int32, device="cuda").fill_(7) for _ in range(nsets)]
        dsts = [torch.empty((nw, n, 4), dtype=torch.int32, device="cuda") for _ in range(nsets)]
        best = None
        for block, waves in shapes:
            pev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(12)]
            for i in range(3):
                stream_probe(srcs[i % nsets], nr, dsts[i % nsets], nw, block, waves, stream=stream)
            for i, (a, b) in enumerate(pev):
                a.record(stream)
                stream_probe(srcs[i % nsets], nr, dsts[i % nsets], nw, block, waves, stream=stream)
                b.record(stream)
            torch.cuda.synchronize()
            pms = sorted(a.elapsed_time(b) for a, b in pev)[len(pev) // 2]                     # timed like the row kernels
            if best is None or pms < best[0]:
                best = (pms, block, waves)
        pms, block, waves = best
        gbs = (nr + nw) * n * 16 / (pms * 1e-3) / 1e9
        out["%dr+%dw" % (nr, nw)] = {"median_ms": round(pms, 5), "achieved_GBps": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4),
                                     "best_shape": {"block_threads": block, "waves_per_cu": waves}}
        del srcs, dsts
    log("reference: flat streams of %d MB, no indirection, best of %d launch shapes each: " % (total_vec * 16 // 1000000, len(shapes))
        + ", ".join("%s %.1f%% (%d threads, %d waves/CU)" % (k, 100 * v["frac"], v["best_shape"]["block_threads"],
                                                            v["best_shape"]["waves_per_cu"]) for k, v in out.items()))
    return out


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=200)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="dsv3")
    ap.add_argument("--level", default=None, help="none|gpu|node (default: the workload's first level)")
    ap.add_argument("--tokens", type=int, default=None,
                    help="send path: tokens per batch instead of the workload's own T (size sweeps; named in config)")
    ap.add_argument("--sets", type=int, default=4, help="rotating buffer sets (cold HBM reads)")
    ap.add_argument("--warm-y", action="store_true",
                    help="combine reads the buffer dispatch wrote in the same step (partly cache-resident) instead of "
                         "an identical one written sets/2 steps earlier")
    ap.add_argument("--path", default="send", choices=["send", "recv", "planner", "table4"],
                    help="send: the headline step (default); recv: the receiver stages of the two-hop exchange; "
                         "planner: dimension selection + expert-swap planner; table4: the K/E/G grid of the paper's Table IV")
    ap.add_argument("--separate-load", action="store_true",
                    help="call hm_expert_load as its own pair of launches instead of letting hm_plan fill the loads")
    ap.add_argument("--separate-cuts", action="store_true",
                    help="planner path: one hm_swap_counts call per group cut instead of one hm_swap_counts_multi")
    ap.add_argument("--monitored", action="store_true",
                    help="planner path: feed the time model with the row counts the receiver-stage plans produce "
                         "(the monitored quantities of Alg.1) next to the fan-in proxy")
    ap.add_argument("--explicit-weights", action="store_true",
                    help="pass the router weights to hm_combine (every wave merges the K slots itself) instead of "
                         "letting it use the weights hm_plan merged")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-table", action="store_true",
                    help="send path: time the named workload only, not the table of all configurations")
    ap.add_argument("--table-steps", type=int, default=30, help="timed steps per row of the configurations table")
    ap.add_argument("--with-transpose", action="store_true", help="also time hm_combine_transpose on the named workload")
    ap.add_argument("--graph", action="store_true",
                    help="send path: capture one step per buffer set in a HIP graph and time graph replays")
    ap.add_argument("--no-warm-leg", action="store_true",
                    help="skip the extra warm (single buffer set) timing and the reference streams, so that a kernel "
                         "trace holds cold launches of the library's kernels only")
    ap.add_argument("--with-f32", action="store_true", help="also time hm_combine_f32 on fp32 rows")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also launch a plain 1 GiB device copy a few times (reference for rocprofv3 FETCH_SIZE/WRITE_SIZE)")
    args = ap.parse_args()

    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (destinations are simulated index partitions; there are "
              "no collectives and no sharding) -- rerun with --gpus 1", file=sys.stderr)
        return 2

    import torch
    from paper_2508_09591_amd import binding as B

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; there is no CPU path", file=sys.stderr)
        return 2
    B.lib()
    torch.cuda.set_device(0)
    if args.path == "recv":
        return run_recv(args)
    if args.path == "planner":
        return run_planner(args)
    if args.path == "table4":
        return run_table4(args)
    return run_send(args)


def run_send(args) -> int:
    import dataclasses
    import torch
    wl, placement_key = get_workload(args.workload)
    label = args.workload
    if args.tokens and args.tokens != wl.T:
        wl = dataclasses.replace(wl, T=args.tokens)
        label = "%s@T=%d" % (label, args.tokens)     # no stored traffic figures for such a size
    level = LEVELS[args.level] if args.level else wl.levels[0]
    head = time_send(wl, level, args.steps, args.warmup, args.sets, label=label, placement_key=placement_key,
                     fused=not args.separate_load, explicit_weights=args.explicit_weights, warm_y=args.warm_y,
                     graph=args.graph, warm_leg=not args.no_warm_leg, transposes=args.with_transpose, with_f32=args.with_f32)
    T, K, H, E = head["T"], head["K"], head["H"], head["E"]
    level_name, c, kern, stream = head["level"], head["c"], head["kern"], head["stream"]
    dominant = max(kern, key=lambda n: kern[n]["avg_ms"])

    # ---- context for the roofline fraction: the runtime's own device-to-device copy of 1 GiB -------
    # (also the known-size launch the rocprofv3 counter runs are scaled by: --calibrate-copy)
    copy_ref = None
    if args.calibrate_copy or not args.no_warm_leg:
        src = torch.empty(1 << 29, dtype=torch.bfloat16, device="cuda").fill_(1.0)      # 1 GiB
        dst = torch.empty_like(src)
        cev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(5)]
        with torch.cuda.stream(stream):
            dst.copy_(src)
            for a, b in cev:
                a.record(stream)
                dst.copy_(src)
                b.record(stream)
        torch.cuda.synchronize()
        cms = sorted(a.elapsed_time(b) for a, b in cev)[len(cev) // 2]
        cgbs = 2 * src.numel() * 2 / (cms * 1e-3) / 1e9
        copy_ref = {"what": "torch copy_ of 1 GiB, device to device (1 read + 1 write stream)", "median_ms": round(cms, 4),
                    "achieved_GBps": round(cgbs, 1), "frac": round(cgbs / HBM_PEAK_GBS, 4)}
        log("reference: plain 1 GiB device copy %.4f ms -> %.1f GB/s = %.1f%% of peak" % (cms, cgbs, 100 * cgbs / HBM_PEAK_GBS))
        del src, dst
    stream_ref = None
    if not args.no_warm_leg:
        stream_ref = flat_stream_references(c, head["alg_bytes"]["hm_dispatch_pack"], head["nsets"], stream)

    # ---- the oracle on this machine's host cores (reported baseline, not the target) ---------------
    cpu = None
    if not args.no_cpu_baseline:
        import oracle
        oracle.build()
        r, x = head["routing"], head["x_host"]
        best = None
        reps = 0
        t_all = time.perf_counter()
        while reps < 12 and (time.perf_counter() - t_all) < 12:      # about 10 s of CPU work
            t1 = time.perf_counter()
            op = oracle.plan(r.topk_ids, r.topk_weights, head["e2r"], head["nodes"], head["rpn"], level)
            oracle.expert_load(r.topk_ids, head["e2r"], head["nodes"], head["rpn"])
            opk = oracle.dispatch_pack(x, op.row_token)
            oracle.combine(opk, r.topk_weights, op.slot_row)
            dt = time.perf_counter() - t1
            best = dt if best is None else min(best, dt)
            reps += 1
        assert op.total_rows == head["total_rows"]
        cpu = {"value": round(T / best, 1), "unit": "tokens/s", "cores": 1, "kind": "oracle",
               "sample": "the whole %s batch (T=%d, level %s), same call sequence, best of %d passes, %.2f s per pass"
                         % (label, T, level_name, reps, best)}
        log("cpu oracle: %.2f s per pass -> %.0f tokens/s on 1 core (%d cores visible)" % (best, T / best, os.cpu_count()))

    # ---- every other configuration of the benchmark set, the same step, fewer repetitions -------
    table = None
    if not args.no_table:
        table = []
        for name, lname in TABLE:
            twl, tkey = get_workload(name)
            if name == label and lname == level_name:
                continue
            big = twl.T >= 32768
            res = time_send(twl, LEVELS[lname], max(5, args.table_steps // (3 if big else 1)), min(args.warmup, 5), args.sets,
                            label=name, placement_key=tkey, host_x=False, transposes=big)
            row = {"workload": name, "level": lname, "T": res["T"], "H": res["H"], "E": res["E"], "K": res["K"],
                   "ranks": "%dx%d" % (res["nodes"], res["rpn"]), "rows_per_token": round(res["c"], 4),
                   "tokens_per_s": round(res["tokens_per_s"], 1), "ms_per_step": round(res["ms_per_step"], 5),
                   "plan_us": round(res["plan_ms"] * 1e3, 2),
                   "dispatch": {k: res["kern"]["hm_dispatch_pack"][k] for k in ("avg_ms", "achieved_GBps", "frac", "traffic")},
                   "combine": {k: res["kern"]["hm_combine"][k] for k in ("avg_ms", "achieved_GBps", "frac", "traffic")},
                   "pair_GBps": round(res["pair_gbs"], 1), "pair_frac": round(res["pair_gbs"] / HBM_PEAK_GBS, 4)}
            row.update(res["extra"])
            table.append(row)
        log("%-13s %-5s %6s %5s %7s %9s %9s %8s %8s %7s" % ("workload", "level", "T", "H", "rows/t", "Mtok/s", "plan us", "disp %", "comb %", "pair %"))
        for row in table:
            log("%-13s %-5s %6d %5d %7.3f %9.2f %9.2f %8.1f %8.1f %7.1f"
                % (row["workload"], row["level"], row["T"], row["H"], row["rows_per_token"], row["tokens_per_s"] / 1e6,
                   row["plan_us"], 100 * row["dispatch"]["frac"], 100 * row["combine"]["frac"], 100 * row["pair_frac"]))

    # ---- the rows built beyond the send path (receiver stages, planner, Table IV grid): short runs of
    # the same code the --path modes run, so that their figures are part of the default record too
    next_rows = None
    if not args.no_table:
        import copy
        sub = copy.copy(args)
        sub.steps, sub.warmup, sub.no_cpu_baseline, sub.monitored, sub.separate_cuts = args.table_steps, min(args.warmup, 5), True, False, False

        def brief(res, keep=("metric", "value", "unit", "ms_per_step", "config", "kernels")):
            out = {k: res[k] for k in keep if k in res}
            out["roofline"] = {k: res["roofline"][k] for k in ("bound", "kernel", "achieved", "peak", "unit", "frac")}
            return out

        next_rows = {}
        sub.workload = "dsv3"
        next_rows["recv"] = brief(run_recv(sub, emit=False))
        for wname in ("skew", "dsv3"):
            sub.workload = wname
            next_rows["planner_" + wname] = brief(run_planner(sub, emit=False, workload=wname))
        t4 = run_table4(sub, emit=False)
        next_rows["table4"] = {"metric": t4["metric"], "grid": [
            {"variant": g["variant"], **{l: {"rows_per_token": g[l]["rows_per_token"], "pair_ms": g[l]["pair_ms"], "frac": g[l]["frac"]}
                                         for l in ("none", "gpu", "node")}} for g in t4["grid"]]}

    result = {
        "metric": "dedup dispatch+combine tokens/s (plan + expert_load + dispatch_pack + combine per step)",
        "expert_load": "separate hm_expert_load call" if args.separate_load else "filled by hm_plan (fused)",
        "combine_weights": "caller's router weights, merged in the kernel" if args.explicit_weights else "merged by hm_plan (row_weight)",
        "launch": "HIP graph replay, one graph per buffer set" if args.graph else "eager launches on one stream",
        "value": round(head["tokens_per_s"], 1),
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(head["ms_per_step"], 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": "%s: T=%d H=%d E=%d top-%d, %d nodes x %d ranks, dedup level %s, identity experts"
                               % (label, T, H, E, K, head["nodes"], head["rpn"], level_name),
                   "rows_per_token": round(c, 4), "buffer_sets": head["nsets"],
                   "combine_input": "same-step buffer (warm)" if args.warm_y else "identical buffer written %d steps earlier (cold)" % head["y_shift"]},
        "roofline": {"bound": "hbm", "kernel": dominant, "achieved": kern[dominant]["achieved_GBps"],
                     "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": kern[dominant]["frac"],
                     "traffic": kern[dominant]["traffic"],
                     "traffic_source": "rocprofv3 FETCH_SIZE + WRITE_SIZE summary under profiles/, taken on these kernel sources"
                                       if kern[dominant]["traffic"] else None},
        "cpu_baseline": cpu,
        "kernels": kern,
        "pair": {"ms": round(head["pair_ms"], 5), "achieved_GBps": round(head["pair_gbs"], 1),
                 "frac": round(head["pair_gbs"] / HBM_PEAK_GBS, 4), "tokens_per_s": round(T / (head["pair_ms"] * 1e-3), 1)},
        "plan_ms": round(head["plan_ms"], 5),
        "event_pair_overhead_ms": round(head["event_overhead_ms"], 5),
        "per_call_timing": "start / stop HIP events around each call on the launch stream; an empty pair already reads "
                           "event_pair_overhead_ms, so a kernel's own duration lies between avg_ms_less_empty_event_pair "
                           "and avg_ms (the kernel traces under profiles/ fall in between); rates use avg_ms",
        "device_copy_reference": copy_ref,
        "flat_stream_reference": stream_ref,
        "expert_load_ms": None if head["expert_load_ms"] is None else round(head["expert_load_ms"], 5),
        "other_calls": head["extra"] or None,
        "configs": table,
        "next_rows": next_rows,
    }
    print(json.dumps(result), flush=True)
    return 0


def run_recv(args, emit=True):
    """Receiver stages of the two-hop exchange (HD2) at the workload's shape, on the rank with local
    index 0 of node 1.  Set-up (untimed) runs the sender path for the 32 source ranks that feed that
    node, so the receiver's inputs have the real size and routing mix:
      stage A (intra-node hop):  hm_plan_mapped(dedup per local rank) + hm_dispatch_pack, and on the
                                 way back hm_combine_mix;
      stage B (local experts):   hm_plan_mapped(one row per slot, expert-contiguous) +
                                 hm_dispatch_pack, and hm_combine_mix after the experts.
    Row contents are random bf16 (they do not affect timing); ids and weights are the real ones."""
    import dataclasses
    import numpy as np
    import torch
    from paper_2508_09591_amd import binding as B
    from paper_2508_09591_amd import workloads as W

    wl = W.WORKLOADS[args.workload]
    T, K, H, E, R, N = wl.T, wl.K, wl.H, wl.E, wl.ranks_per_node, wl.nodes
    node = 1 % N
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    e2r = W.contiguous_placement(E, wl.G)
    e2r_d = dev(e2r)
    stream = torch.cuda.Stream()

    def pack_meta(plan, t, rows):                     # ids / weights travel as rows of 2K 2-byte units
        out = torch.empty((rows, 2 * K), dtype=torch.bfloat16, device="cuda")
        B.hm_dispatch_pack(t.view(torch.bfloat16).view(-1, 2 * K), plan, out, stream=stream)
        return out

    t0 = time.time()
    with torch.cuda.stream(stream):
        recv_ids, recv_w = [], []                     # per receiver (node, r): rows arriving from the N source nodes
        for r in range(R):
            parts_i, parts_w = [], []
            for n in range(N):
                rt = W.make_routing(dataclasses.replace(wl, seed=1000 + n * R + r))
                ids_d, w_d = dev(rt.topk_ids), dev(rt.topk_weights)
                p1 = B.hm_plan(ids_d, w_d, e2r_d, N, R, B.HM_DEDUP_NODE, stream=stream)
                st, tot = B.hm_plan_status(p1, stream=stream)
                assert st == 0
                off = p1.dest_offset[:N + 1].cpu().numpy()
                a, b = int(off[node]), int(off[node + 1])
                parts_i.append(pack_meta(p1, ids_d, tot)[a:b].contiguous().view(torch.int32).view(-1, K))
                parts_w.append(pack_meta(p1, w_d, tot)[a:b].contiguous().view(torch.float32).view(-1, K))
            recv_ids.append(torch.cat(parts_i).contiguous())
            recv_w.append(torch.cat(parts_w).contiguous())
        # stage A on every receiver of the node (needed to build stage B's input for local rank 0)
        dmA = torch.empty(E, dtype=torch.int32, device="cuda")
        ndA = torch.empty(1, dtype=torch.int32, device="cuda")
        B.hm_recv_dest_map(e2r_d, N, R, node * R, B.HM_RECV_INTRA_NODE, dmA, ndA, stream=stream)
        b_ids, b_w = [], []
        planA = None
        for r in range(R):
            pa = B.hm_plan_mapped(recv_ids[r], recv_w[r], dmA, R, True, stream=stream)
            st, tot = B.hm_plan_status(pa, stream=stream)
            assert st == 0
            off = pa.dest_offset[:R + 1].cpu().numpy()
            b_ids.append(pack_meta(pa, recv_ids[r], tot)[int(off[0]):int(off[1])].contiguous().view(torch.int32).view(-1, K))
            b_w.append(pack_meta(pa, recv_w[r], tot)[int(off[0]):int(off[1])].contiguous().view(torch.float32).view(-1, K))
            if r == 0:
                planA, rowsA_out = pa, tot
        idsA, wA = recv_ids[0], recv_w[0]
        idsB, wB = torch.cat(b_ids).contiguous(), torch.cat(b_w).contiguous()
        dmB = torch.empty(E, dtype=torch.int32, device="cuda")
        ndB = torch.empty(1, dtype=torch.int32, device="cuda")
        B.hm_recv_dest_map(e2r_d, N, R, node * R, B.HM_RECV_LOCAL_EXPERTS, dmB, ndB, stream=stream)
        n_local = int(ndB.item())
        planB = B.hm_plan_mapped(idsB, wB, dmB, n_local, False, stream=stream)
        st, rowsB_out = B.hm_plan_status(planB, stream=stream)
        assert st == 0
    rowsA_in, rowsB_in = idsA.shape[0], idsB.shape[0]
    log("set-up %.1f s; stage A: %d rows in -> %d rows out (x%.2f); stage B: %d rows in -> %d expert rows (x%.2f, %d local experts)"
        % (time.time() - t0, rowsA_in, rowsA_out, rowsA_out / rowsA_in, rowsB_in, rowsB_out, rowsB_out / rowsB_in, n_local))

    nsets = max(1, args.sets)
    mk = lambda rows: [torch.randn((rows, H), dtype=torch.float32, device="cuda").to(torch.bfloat16) for _ in range(nsets)]
    inA, outA, backA = mk(rowsA_in), mk(rowsA_out), mk(rowsA_in)
    inB, outB, backB = mk(rowsB_in), mk(rowsB_out), mk(rowsB_in)

    calls = [
        ("A.hm_plan_mapped", lambda s: B.hm_plan_mapped(idsA, wA, dmA, R, True, plan=planA, stream=stream), 0),
        ("A.hm_dispatch_pack", lambda s: B.hm_dispatch_pack(inA[s], planA, outA[s], stream=stream), (rowsA_in + rowsA_out) * 2 * H),
        ("A.hm_combine_mix", lambda s: B.hm_combine_mix(outA[(s + nsets // 2) % nsets], None, planA, backA[s], stream=stream), (rowsA_in + rowsA_out) * 2 * H),
        ("B.hm_plan_mapped", lambda s: B.hm_plan_mapped(idsB, wB, dmB, n_local, False, plan=planB, stream=stream), 0),
        ("B.hm_dispatch_pack", lambda s: B.hm_dispatch_pack(inB[s], planB, outB[s], stream=stream), (rowsB_in + rowsB_out) * 2 * H),
        ("B.hm_combine_mix", lambda s: B.hm_combine_mix(outB[(s + nsets // 2) % nsets], None, planB, backB[s], stream=stream), (rowsB_in + rowsB_out) * 2 * H),
    ]

    def step(i, ev=None):
        s = i % nsets
        for j, (_, fn, _) in enumerate(calls):
            if ev: ev[j].record(stream)
            fn(s)
        if ev: ev[len(calls)].record(stream)

    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()
    t_begin = time.perf_counter()
    for i in range(args.steps):
        step(i)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t_begin
    events = [[torch.cuda.Event(enable_timing=True) for _ in range(len(calls) + 1)] for _ in range(args.steps)]
    for i in range(args.steps):
        step(i, events[i])
    torch.cuda.synchronize()
    kern = {}
    for j, (name, _, nbytes) in enumerate(calls):
        ms = sum(e[j].elapsed_time(e[j + 1]) for e in events) / args.steps
        kern[name] = {"avg_ms": round(ms, 5)}
        if nbytes:
            gbs = nbytes / (ms * 1e-3) / 1e9
            kern[name].update({"alg_bytes": int(nbytes), "achieved_GBps": round(gbs, 1), "frac": round(gbs / HBM_PEAK_GBS, 4)})
        log("%-20s %.4f ms %s" % (name, ms, ("%.0f GB/s (%.1f%%)" % (kern[name]["achieved_GBps"], 100 * kern[name]["frac"])) if nbytes else ""))
    dominant = max((n for n in kern if "frac" in kern[n]), key=lambda n: kern[n]["avg_ms"])
    ms_per_step = elapsed * 1e3 / args.steps
    result = {
        "metric": "HD2 receiver stages (intra-node re-dedup + local-expert expand, forward and normalised merge back): received rows/s",
        "value": round(rowsA_in / (ms_per_step * 1e-3), 1), "unit": "rows/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 5), "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": "%s receiver: rank 0 of node %d, %d nodes x %d ranks, H=%d; stage A %d->%d rows, stage B %d->%d rows"
                               % (wl.name, node, N, R, H, rowsA_in, rowsA_out, rowsB_in, rowsB_out), "buffer_sets": nsets},
        "roofline": {"bound": "hbm", "kernel": dominant, "achieved": kern[dominant]["achieved_GBps"], "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": kern[dominant]["frac"], "traffic": None},
        "cpu_baseline": None, "kernels": kern,
    }
    if not emit:
        return result
    print(json.dumps(result), flush=True)
    return 0


def run_planner(args, emit=True, workload=None):
    """The per-iteration planner work of Sections III-C and IV on the device: per-level counts,
    the time model and d*, the swap tensor Z for every level of a 4-level hierarchy, and the
    selection of the best expert pair (gamma = 10).  Default workload here: skew (config 4)."""
    import numpy as np
    import torch
    from paper_2508_09591_amd import binding as B
    from paper_2508_09591_amd import workloads as W

    wl = W.WORKLOADS[workload or (args.workload if args.workload != "dsv3" or "--workload" in sys.argv else "skew")]
    r = W.make_routing(wl)
    e2r = r.extras.get("expert_to_rank_swapped", r.expert_to_rank)
    T, K, E, G, H = wl.T, wl.K, wl.E, wl.G, wl.H
    U = [1, wl.nodes, wl.nodes * 2, wl.nodes * 4]
    U = [u for u in U if G % u == 0 and u <= G]
    D = len(U)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ids_d, e2r_d = dev(r.topk_ids), dev(e2r)
    stream = torch.cuda.Stream()
    ai, bi = [0, 4.97e-1, 3.01e-1, 1.49e-1][:D], [0, 5.29e-7, 1.17e-7, 2.06e-8][:D]     # the paper's Fig.9 fit
    aa, ba = [7.22e-1, 5.71e-1, 1.14e-1, 2.04e-1][:D], [5.70e-7, 1.27e-7, 2.63e-8, 1.64e-8][:D]
    own = torch.zeros((D, 64), dtype=torch.int32, device="cuda")
    times = torch.zeros(4, dtype=torch.float64, device="cuda")
    best_d = torch.zeros(1, dtype=torch.int32, device="cuda")
    cuts = sorted(set(U[1:] + [G]))
    Z = {u: torch.empty((E, E, u), dtype=torch.int32, device="cuda") for u in cuts}
    ws = {u: torch.empty(int(B.lib().hm_swap_workspace_bytes(T, K, E, u)) // 4 + 4, dtype=torch.int32, device="cuda") for u in cuts}
    ws_multi = None
    if not args.separate_cuts:
        import ctypes
        nga = (ctypes.c_int32 * len(cuts))(*cuts)
        ws_multi = torch.empty(int(B.lib().hm_swap_multi_workspace_bytes(T, K, E, G, len(cuts), nga)) // 4 + 4,
                               dtype=torch.int32, device="cuda")
    Q = torch.empty((E, E), dtype=torch.float64, device="cuda")
    bp = torch.zeros(2, dtype=torch.int32, device="cuda")
    bt = torch.zeros(1, dtype=torch.float64, device="cuda")
    ws_sel = torch.empty(int(B.lib().hm_swap_select_workspace_bytes(E)) // 8 + 2, dtype=torch.float64, device="cuda")
    fan_in = torch.tensor(U, dtype=torch.int32, device="cuda")[:, None]
    si = [0.0] + [float(U[i - 1]) for i in range(1, D)]

    def step(ev=None):
        if ev: ev[0].record(stream)
        B.hm_group_counts(ids_d, e2r_d, G, [G] + U[1:], own, stream=stream)
        if ev: ev[1].record(stream)
        with torch.cuda.stream(stream):                 # harness: counts before Intra-level-l = own counts x fan-in
            p_intra = (own[0:1] * fan_in).contiguous()
        B.hm_alltoall_times(U, G, H, 2.0, own, p_intra, ai, bi, aa, ba, times, best_d, stream=stream)
        if ev: ev[2].record(stream)
        if args.separate_cuts:
            for u in cuts:
                B.hm_swap_counts(ids_d, e2r_d, G, u, Z[u], workspace=ws[u], stream=stream)
        else:                                            # all cuts in one pass over the tokens
            B.hm_swap_counts_multi(ids_d, e2r_d, G, cuts, [Z[u] for u in cuts], workspace=ws_multi, stream=stream)
        if ev: ev[3].record(stream)
        B.hm_swap_select(U, G, H, 2.0, [None] + [Z[u] for u in U[1:]], Z[G], si, float(U[D - 1]), ai, bi, aa[D - 1],
                         ba[D - 1], 10.0, Q, bp, bt, workspace=ws_sel, stream=stream)
        if ev: ev[4].record(stream)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
    events = [[torch.cuda.Event(enable_timing=True) for _ in range(5)] for _ in range(args.steps)]
    for i in range(args.steps):
        step(events[i])
    torch.cuda.synchronize()
    names = ["hm_group_counts", "hm_alltoall_times",
             ("hm_swap_counts x%d" if args.separate_cuts else "hm_swap_counts_multi (%d cuts)") % len(cuts), "hm_swap_select"]
    kern = {n: round(sum(e[j].elapsed_time(e[j + 1]) for e in events) / args.steps, 5) for j, n in enumerate(names)}
    log("planner on %s (T=%d K=%d E=%d G=%d, U=%s): %.4f ms per step; " % (wl.name, T, K, E, G, U, ms_per_step)
        + ", ".join("%s %.4f ms" % kv for kv in kern.items()))
    log("d* = %d, t_d = %s; best swap %s -> %.4f vs %.4f without a swap"
        % (int(best_d.item()), np.round(times.cpu().numpy()[:D], 4).tolist(), tuple(bp.cpu().numpy().tolist()),
           float(bt.item()), float(Q[0, 0].item())))
    monitored = None
    if args.monitored:
        monitored = monitored_dimension_choice(wl, e2r, ai, bi, aa, ba, stream)
    cpu = None
    if not args.no_cpu_baseline:
        import oracle
        oracle.build()
        t1 = time.perf_counter()
        oracle.group_counts(r.topk_ids, e2r, G, [G] + U[1:])
        zs = {u: oracle.swap_counts(r.topk_ids, e2r, G, u, "incremental")[0] for u in cuts}
        oracle.swap_select(U, G, H, 2.0, [None] + [zs[u] for u in U[1:]], zs[G], si, float(U[D - 1]), ai, bi, aa[D - 1],
                           ba[D - 1], 10.0)
        dt = time.perf_counter() - t1
        cpu = {"value": round(T / dt, 1), "unit": "tokens/s", "cores": 1, "kind": "oracle",
               "sample": "the whole %s batch once (incremental Z update for %d cuts + selection), %.2f s" % (wl.name, len(cuts), dt)}
        log("cpu oracle: %.2f s" % dt)
    swap_ms = kern[names[2]]
    # The co-occurrence tables are matrix products over 0/1 indicator tiles in FP4 (E <= 256): per cut C = A^T S (rows x
    # columns x T) and CG = S^T M (columns x 32 ceil(ng/32) x T), rows and columns of C padded to whole tiles and panels.  Their
    # dense operation count against the FP4 MFMA peak is what the line reports; the products themselves are a small part of
    # the call (filling the tiles, barriers and LDS latency, and two short launches, set its time).
    rows, panel = 32 * ((E + 31) // 32), 64 if E > 128 else 32
    cols = panel * ((E + panel - 1) // panel)
    dense_ops = sum(2 * cols * (rows + 32 * ((u + 31) // 32)) * T for u in cuts) if E <= 256 else 0
    peak_ops = 10.0e15
    result = {"metric": "planner (counts + d* + swap tensor Z + best pair) tokens/s", "value": round(T / (ms_per_step * 1e-3), 1),
              "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_per_step, 5),
              "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int32", "data": "synthetic",
              "config": {"workload": "%s: T=%d K=%d E=%d G=%d, hierarchy U=%s, gamma=10" % (wl.name, T, K, E, G, U)},
              "roofline": {"bound": "mfma", "kernel": "hm_swap_counts_multi (swap_cooc + swap_pairs)",
                           "achieved": round(dense_ops / (swap_ms * 1e-3) / 1e12, 3), "peak": round(peak_ops / 1e12, 1),
                           "unit": "FP4 TFLOP/s (dense products of the 0/1 indicator tiles; peak: MI355X FP4 MFMA, dense)",
                           "frac": round(dense_ops / (swap_ms * 1e-3) / peak_ops, 5), "traffic": None,
                           "dense_ops_per_call": dense_ops,
                           "note": "latency-bound: seven or eight short launches per planner step over a few hundred KiB of input; in the "
                                   "matrix kernel the products are a small part of the time, loads, marks and stores of the tables "
                                   "the rest"},
              "cpu_baseline": cpu, "kernels": kern, "monitored_counts": monitored}
    if not emit:
        return result
    print(json.dumps(result), flush=True)
    return 0


def monitored_dimension_choice(wl, e2r, ai, bi, aa, ba, stream):
    """Alg.1 for the two-dimensional exchange with the counts it monitors instead of the fan-in
    proxy: the inter-node hop of the N same-local-index source ranks is run on the device (each
    with its own seeded routing), the receiver's intra-node plan gives the per-GPU counts of the
    tokens it holds after that hop, p^(2,G), and hm_alltoall_times takes those dest_count vectors
    straight from device memory.  Returns both sets of times and d*."""
    import dataclasses
    import numpy as np
    import torch
    from paper_2508_09591_amd import binding as B
    from paper_2508_09591_amd import workloads as W

    N, R, G, K, E = wl.nodes, wl.ranks_per_node, wl.G, wl.K, wl.E
    node, local = 1 % N, 0
    me = node * R + local
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    e2r_d = dev(e2r)
    parts_i, parts_w, own = [], [], None
    with torch.cuda.stream(stream):
        for n in range(N):
            rt = W.make_routing(dataclasses.replace(wl, seed=1000 + n * R + local))
            ids_d, w_d = dev(rt.topk_ids), dev(rt.topk_weights)
            if n == node:
                own = (ids_d, w_d)
            p1 = B.hm_plan(ids_d, w_d, e2r_d, N, R, B.HM_DEDUP_NODE, stream=stream)
            st, tot = B.hm_plan_status(p1, stream=stream)
            assert st == 0
            off = p1.dest_offset[:N + 1].cpu().numpy()
            a, b = int(off[node]), int(off[node + 1])
            for t, parts, dt in ((ids_d, parts_i, torch.int32), (w_d, parts_w, torch.float32)):
                rows = torch.empty((tot, 2 * K), dtype=torch.bfloat16, device="cuda")
                B.hm_dispatch_pack(t.view(torch.bfloat16).view(-1, 2 * K), p1, rows, stream=stream)
                parts.append(rows[a:b].contiguous().view(dt).view(-1, K))
        rid, rw = torch.cat(parts_i).contiguous(), torch.cat(parts_w).contiguous()
        dmA = torch.empty(E, dtype=torch.int32, device="cuda")
        ndA = torch.empty(1, dtype=torch.int32, device="cuda")
        B.hm_recv_dest_map(e2r_d, N, R, me, B.HM_RECV_INTRA_NODE, dmA, ndA, stream=stream)
        planA = B.hm_plan_mapped(rid, rw, dmA, R, True, stream=stream)
        plan_gpu = B.hm_plan(own[0], own[1], e2r_d, N, R, B.HM_DEDUP_GPU, stream=stream)
        plan_node = B.hm_plan(own[0], own[1], e2r_d, N, R, B.HM_DEDUP_NODE, stream=stream)
        p_inter = torch.zeros((2, 64), dtype=torch.int32, device="cuda")
        p_intra = torch.zeros((2, 64), dtype=torch.int32, device="cuda")
        p_inter[1, :N] = plan_node.dest_count[:N]
        p_intra[0, :G] = plan_gpu.dest_count[:G]
        p_intra[1, :R] = planA.dest_count[:R]            # the monitored counts
        p_proxy = p_intra.clone()
        p_proxy[1, :G] = plan_gpu.dest_count[:G] * N     # the proxy: own per-GPU counts times the fan-in
        times = torch.zeros(4, dtype=torch.float64, device="cuda")
        best = torch.zeros(1, dtype=torch.int32, device="cuda")
        out = {}
        for name, pa in (("monitored", p_intra), ("fan_in_proxy", p_proxy)):
            B.hm_alltoall_times([1, N], G, wl.H, 2.0, p_inter, pa, ai[:2], bi[:2], aa[:2], ba[:2], times, best, stream=stream)
            torch.cuda.synchronize()
            out[name] = {"t_d": [round(float(x), 6) for x in times.cpu().numpy()[:2]], "d_star": int(best.item()),
                         "max_p2G": int(pa[1].max().item())}
    out["what"] = ("two-dimensional exchange U=[1,%d] seen from rank %d: received rows %d -> %d after the intra-node re-dedup"
                   % (N, me, rid.shape[0], int(planA.dest_count[:R].sum().item())))
    log("Alg.1 with monitored counts: %s; fan-in proxy: %s" % (out["monitored"], out["fan_in_proxy"]))
    return out


def run_table4(args, emit=True):
    """The K / E / G grid of the paper's Table IV on the Qwen3-shaped layer: rows per token at the
    three dedup levels (what the deduplication saves) and the dispatch+combine rate at each."""
    import numpy as np
    import torch
    from paper_2508_09591_amd import binding as B
    from paper_2508_09591_amd import workloads as W

    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    stream = torch.cuda.Stream()
    table = []
    for wl in W.table4_variants():
        T, K, H, E = wl.T, wl.K, wl.H, wl.E
        r = W.make_routing(wl)
        ids_d, w_d, e2r_d = dev(r.topk_ids), dev(r.topk_weights), dev(r.expert_to_rank)
        x = torch.randn((T, H), dtype=torch.float32, device="cuda").to(torch.bfloat16)
        row = {"variant": wl.name, "K": K, "E": E, "G": wl.G}
        for level, lname in ((0, "none"), (1, "gpu"), (2, "node")):
            plan = B.hm_plan(ids_d, w_d, e2r_d, wl.nodes, wl.ranks_per_node, level, stream=stream)
            st, total = B.hm_plan_status(plan, stream=stream)
            assert st == 0
            nsets = 4
            xs = [x.clone() for _ in range(nsets)]
            packs = [torch.empty((total, H), dtype=torch.bfloat16, device="cuda") for _ in range(nsets)]
            outs = [torch.empty((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(nsets)]
            for s_ in range(nsets):
                B.hm_dispatch_pack(xs[s_], plan, packs[s_], stream=stream)

            def pair(i):
                s_ = i % nsets
                B.hm_dispatch_pack(xs[s_], plan, packs[s_], stream=stream)
                B.hm_combine(packs[(s_ + 2) % nsets], None, plan, outs[s_], stream=stream)

            for i in range(args.warmup):
                pair(i)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record(stream)
            for i in range(args.steps):
                pair(i)
            e1.record(stream)
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / args.steps
            nbytes = 2 * (T + total) * H * 2
            row[lname] = {"rows_per_token": round(total / T, 4), "pair_ms": round(ms, 5),
                          "GBps": round(nbytes / (ms * 1e-3) / 1e9, 1), "frac": round(nbytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS, 4)}
        row["bytes_saved_vs_none"] = {l: round(1 - (1 + row[l]["rows_per_token"]) / (1 + row["none"]["rows_per_token"]), 4)
                                      for l in ("gpu", "node")}
        table.append(row)
        log("%-5s K=%-2d E=%-3d G=%-2d  rows/token none %.2f gpu %.3f node %.3f | pair ms %.4f / %.4f / %.4f | %% of peak %.1f / %.1f / %.1f"
            % (wl.name, K, E, wl.G, row["none"]["rows_per_token"], row["gpu"]["rows_per_token"], row["node"]["rows_per_token"],
               row["none"]["pair_ms"], row["gpu"]["pair_ms"], row["node"]["pair_ms"],
               100 * row["none"]["frac"], 100 * row["gpu"]["frac"], 100 * row["node"]["frac"]))
    ref = next(r_ for r_ in table if r_["variant"] == "K8")
    result = {"metric": "dispatch+combine over the Table IV grid (Qwen3 shape): tokens/s at K=8, E=128, G=32, node level",
              "value": round(8192 / (ref["node"]["pair_ms"] * 1e-3), 1), "unit": "tokens/s", "n_gpus": 1, "steps": args.steps,
              "warmup": args.warmup, "ms_per_step": ref["node"]["pair_ms"], "higher_is_better": True, "scaling": "weak",
              "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
              "config": {"workload": "qwen3 shape (T=8192, H=2048), K in {6,8,10}, E in {64,128,256}, G in {8,16,32}"},
              "roofline": {"bound": "hbm", "kernel": "hm_dispatch_pack+hm_combine", "achieved": ref["node"]["GBps"],
                           "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": ref["node"]["frac"], "traffic": None},
              "cpu_baseline": None, "grid": table}
    if not emit:
        return result
    print(json.dumps(result), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
