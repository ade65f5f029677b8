#!/usr/bin/env python3
"""Benchmark of the dynamically gated MoE layer forward on one MI355X.

A step is one moe_layer_forward call (gate GEMM, softmax/top-k, counts + scan + stable
permutation, dispatch, grouped expert FFN, combine) over one batch of synthetic tokens, all
inputs resident in HBM before the timed region starts.  Prints ONE JSON line:
tokens/s of the whole layer, the roofline figures of the dominant kernel (live HIP-event
timing on the stream the kernels run on), a per-kernel breakdown, and the CPU oracle timed
on the host cores as a reported baseline.

The headline workload is `skewed_large`, the largest of the five (T 65536, E 128, 2048 -> 8192, Zipf 1.2);
the other four are reported under "also".

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config skewed_large] [--also lm,...]
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

HBM_PEAK_GBS = 8000.0         # MI355X HBM3E
MFMA_BF16_PEAK_TFLOPS = 2500.0  # dense bf16 MFMA
MFMA_F32_PEAK_TFLOPS = 157.3  # dense fp32 MFMA (the fp32 GEMMs run on v_mfma_f32_32x32x2_f32)


# Every timed block is preceded by a fixed, untimed pre-conditioning phase of this many seconds of the same
# steps (on top of --warmup): the device's clocks and power state settle over a few hundred milliseconds of
# load, and a short warm-up otherwise leaves the first timed steps slow (20 steps after 5 warm-up steps read
# up to 17 % slower than 200 after 50).
PRECONDITION_SECONDS = 1.0

# Last-level cache of the device (the 256 MB cache in front of HBM): a workload whose weights fit keeps them
# there between steps, so such a workload is also run "cold", rotating through enough copies of its weights.
LAST_LEVEL_CACHE_BYTES = 256 << 20


def profile_kernel_name(kernel: str):
    """bench name of a kernel row of profiles/moe_layer_forward_*.txt (None = not one of the layer's steps)."""
    k = kernel.strip()
    if k.startswith("gemm_bf16_kernel<") or k.startswith("gemm_f32"):
        args = [a.strip() for a in k[k.index("<") + 1:].rstrip(">").split(",")]
        if k.startswith("gemm_bf16_kernel<"):
            out_f32, relu, grouped = args[4] == "true", args[5] == "true", args[6] == "true"
            if len(args) > 10 and args[-1] != "0":
                return None  # quantised weights (the weight_formats runs), not the bf16 layer
        else:  # gemm_f32_*<[waves,] RELU, GROUPED, ...>
            if k.startswith("gemm_f32_wave_kernel<"):
                args = args[1:]
            out_f32, relu, grouped = False, args[0] == "true", args[1] == "true"
        if not grouped:
            return "gate_gemm" if (out_f32 or k.startswith("gemm_f32")) else None
        return "expert_gemm1" if relu else "expert_gemm2"
    if k.startswith("gemm_ring_kernel<"):  # <RELU, RAGGED, weight storage, TURNED>
        if [a.strip() for a in k[k.index("<") + 1:].rstrip(">").split(",")][2:3] not in ([], ["0"]):
            return None  # quantised weights
        return "expert_gemm1" if k[k.index("<") + 1:].startswith("true") else "expert_gemm2"
    if k.startswith("gemm_stream_kernel<"):  # <weight storage, RELU, ...>
        args = [a.strip() for a in k[k.index("<") + 1:].rstrip(">").split(",")]
        return None if args[0] != "0" else "expert_gemm1" if args[1] == "true" else "expert_gemm2"
    for prefix, name in (("gate_topk_", "gate_topk"), ("topk_kernel", "topk"), ("route_", "route"),
                         ("dispatch_kernel", "dispatch"), ("combine_kernel", "combine"), ("tile_map_kernel", "tile_map")):
        if k.startswith(prefix):
            return name
    return None


def traffic_from_profile(workload: str, profiles_dir: str = None):
    """HBM-side bytes per launch of every kernel of the layer, from the committed rocprofv3 counter summary
    profiles/moe_layer_forward_<workload>.txt: the FETCH_SIZE and WRITE_SIZE sections (KiB per dispatch, two
    --pmc runs), each scaled by what the same counter reads for the 1 GiB-read + 1 GiB-write calibration kernel
    of the same run (the row of torch's elementwise add).  A step made of several launches (the routing
    kernels) is the sum over them.  {} when there is no summary for the workload."""
    path = os.path.join(profiles_dir or os.path.join(ROOT, "profiles"), "moe_layer_forward_%s.txt" % workload)
    if not os.path.exists(path):
        return {}
    section, rows = None, {"FETCH_SIZE": {}, "WRITE_SIZE": {}}
    for line in open(path):
        if line.startswith("== "):
            section = line[3:].split()[0]
            continue
        if section in rows and " KiB" in line and " n=" in line:
            kernel = line[:line.index(" n=")].strip()
            rows[section][kernel] = rows[section].get(kernel, 0.0) + float(line.rsplit("KiB", 1)[0].split()[-1])
    out = {}
    factors = {}
    for sec in rows:
        calib = [v for k, v in rows[sec].items() if "FunctorOnSelf_add<int>" in k]
        if not calib:
            return {}
        factors[sec] = (1 << 20) / calib[0]   # the calibration kernel moves 1 GiB = 2^20 KiB each way
    for sec in rows:
        for kernel, kib in rows[sec].items():
            name = profile_kernel_name(kernel)
            if name:
                out[name] = out.get(name, 0.0) + factors[sec] * kib * 1024.0
    return {k: int(round(v)) for k, v in out.items()}


def kernel_models(w, counts):
    """Algorithmic bytes / flops per launch of every kernel of the layer (what the method
    itself must move or compute, independent of how the kernels are written)."""
    b = 2 if w.dtype == "bf16" else 4
    T, D, F, E, k = w.T, w.D, w.F, w.E, w.k
    N = k * T
    e_active = int((counts > 0).sum())
    m = {}
    m["gate_gemm"] = dict(bytes=T * D * b + E * D * b + 4 * T * E, flops=2 * T * D * E)
    m["topk"] = dict(bytes=4 * T * E + 8 * T * k, flops=0)
    # gate GEMM with the top-k decision (and the tile histograms) in its epilogue: x and Wg in, indices and
    # weights out; the logits stay in registers, so their 2 x 4*T*E bytes are NOT counted here
    m["gate_topk"] = dict(bytes=T * D * b + E * D * b + 8 * T * k + 4 * ((T + 31) // 32) * E, flops=2 * T * D * E)
    # a decoder step's selection is made in the routing launch: the logits in, the weights out as well
    fused_topk = m["topk"]["bytes"] if T <= 64 and E % 4 == 0 else 0
    m["route"] = dict(bytes=12 * N + 4 * E + fused_topk, flops=0)
    m["dispatch"] = dict(bytes=T * D * b + N * D * b + 4 * N, flops=0)
    m["expert_gemm1"] = dict(bytes=e_active * F * D * b + N * D * b + N * F * b, flops=2 * N * D * F)
    m["expert_gemm2"] = dict(bytes=e_active * F * D * b + N * F * b + N * D * b, flops=2 * N * D * F)
    m["combine"] = dict(bytes=N * D * b + T * D * b + 8 * N, flops=0)
    m["tile_map"] = dict(bytes=8 * E, flops=0)
    return m


def roofline_entry(name, model, ms, dtype):
    """Which roof bounds the kernel and the achieved fraction of it."""
    secs = ms * 1e-3
    peak_tf = MFMA_BF16_PEAK_TFLOPS if dtype == "bf16" else MFMA_F32_PEAK_TFLOPS
    t_mem = model["bytes"] / (HBM_PEAK_GBS * 1e9)
    t_alu = model["flops"] / (peak_tf * 1e12)
    if t_alu > t_mem:
        ach = model["flops"] / secs / 1e12
        return dict(kernel=name, bound="mfma", achieved=ach, peak=peak_tf,
                    unit="TFLOP/s", frac=ach / peak_tf, traffic=None, avg_ms=ms)
    ach = model["bytes"] / secs / 1e9
    return dict(kernel=name, bound="hbm", achieved=ach, peak=HBM_PEAK_GBS, unit="GB/s", frac=ach / HBM_PEAK_GBS,
                traffic=None, avg_ms=ms)


def precondition(step, seconds=PRECONDITION_SECONDS):
    """Untimed steps for a fixed wall time, so that every timed block starts from the same clock / power state
    whatever --warmup says."""
    import torch
    t0 = time.perf_counter()
    n = 0
    while time.perf_counter() - t0 < seconds:
        for _ in range(4):
            step()
        torch.cuda.synchronize()
        n += 4
    return n


def timed_block(step, steps):
    """EXACTLY `steps` steps between synchronisations; the larger of wall clock and stream events."""
    import torch
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    ev0.record()
    for _ in range(steps):
        step()
    ev1.record()
    torch.cuda.synchronize()
    wall_ms = (time.perf_counter() - t0) * 1e3
    return max(wall_ms, ev0.elapsed_time(ev1)) / steps


def run_config(name, steps, warmup, profile_steps=10, cold_copies=0):
    import numpy as np
    import torch
    from paper_2303_06182_amd import binding, workloads as wl

    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w, device="cuda")
    layer = binding.MoeLayer(w.T, w.D, w.F, w.E, w.k, w.dtype)
    y = torch.empty((w.T, w.D), dtype=w.torch_dtype, device="cuda")
    routing = layer.empty_routing(w.T)
    # the timed step asks for the per-expert counts only (the kernel models below need them): the method itself
    # needs neither the logits nor any other routing array outside the library's workspace
    layer.moe_layer_forward(inp["x"], inp["wg"], inp["w1"], inp["w2"], inp["gate_bias"], y=y, routing_out=routing)
    counts_only = dict(counts=routing["counts"])

    def step():
        layer.moe_layer_forward(inp["x"], inp["wg"], inp["w1"], inp["w2"], inp["gate_bias"], y=y,
                                routing_out=counts_only)

    pre_steps = precondition(step)
    for _ in range(warmup):
        step()
    ms_per_step = timed_block(step, steps)
    counts = routing["counts"].cpu().numpy()

    # the spread behind the mean: the same steps again, each between an event pair of its own
    pairs = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    for a, b in pairs:
        a.record()
        step()
        b.record()
    torch.cuda.synchronize()
    each = sorted(a.elapsed_time(b) for a, b in pairs)
    step_ms = dict(median=each[len(each) // 2], min=each[0], max=each[-1], n=len(each))
    # bytes one step must touch (expert weights with rows + activations): against the 256 MB last-level
    # cache this says whether a step can find its weights cached from the step before
    es = 2 if w.dtype == "bf16" else 4
    weight_bytes = int((counts > 0).sum()) * 2 * w.D * w.F * es
    working_set = weight_bytes + w.T * w.k * (2 * w.D + w.F) * es

    # a workload whose weights fit the last-level cache: the same steps again, every step on the next of
    # `cold_copies` copies of the weights, so that no step finds its weights cached
    cold = None
    if cold_copies > 1:
        copies = [(inp["w1"], inp["w2"], inp["wg"])] + [(inp["w1"].clone(), inp["w2"].clone(), inp["wg"].clone())
                                                       for _ in range(cold_copies - 1)]
        turn = [0]

        def cold_step():
            w1, w2, wg = copies[turn[0] % len(copies)]
            turn[0] += 1
            layer.moe_layer_forward(inp["x"], wg, w1, w2, inp["gate_bias"], y=y, routing_out=counts_only)

        precondition(cold_step)
        cold = dict(ms_per_step=timed_block(cold_step, steps), weight_copies=cold_copies,
                    rotated_bytes=cold_copies * weight_bytes)
        cold["tokens_per_s"] = w.T / (cold["ms_per_step"] * 1e-3)
        del copies

    # per-kernel durations: HIP events recorded by the library around every launch, on the same stream
    acc = {}
    for _ in range(profile_steps):
        layer.moe_profile_begin()
        step()
        for kname, ms in layer.moe_profile_end():
            acc.setdefault(kname, []).append(ms)
    # the fused call folds the dispatch into the first expert GEMM's row addressing where it can;
    # the dispatch step as an entry point of its own is then timed beside it
    standalone = set()
    if "dispatch" not in acc:
        for _ in range(profile_steps):
            layer.moe_profile_begin()
            xp = layer.moe_dispatch(inp["x"], routing["dst_row"])
            for kname, ms in layer.moe_profile_end():
                acc.setdefault(kname, []).append(ms)
        del xp
        standalone.add("dispatch")
    # what an event pair around nothing reads: subtracted from every record (it is a third to a half of what
    # the events show for the kernels of 5 to 20 us)
    overhead_ms = float(np.median(acc.pop("event_pair_overhead", [0.0])))
    kernels = {}
    models = kernel_models(w, counts)
    traffic = traffic_from_profile(name)
    for kname, v in acc.items():
        raw = float(np.mean(v))
        ms = max(raw - overhead_ms, 0.25 * raw)
        kernels[kname] = roofline_entry(kname, models[kname], ms, w.dtype)
        kernels[kname]["event_ms"] = raw
        kernels[kname]["traffic"] = traffic.get(kname)
        kernels[kname]["algorithmic_bytes"] = models[kname]["bytes"]
        kernels[kname]["algorithmic_flops"] = models[kname]["flops"]
        if kname in standalone:
            kernels[kname]["in_fused_call"] = False  # measured through its own entry point, not part of ms_per_step
    dominant = max((r for r in kernels.values() if r.get("in_fused_call", True)), key=lambda r: r["avg_ms"])
    res = dict(workload=name, T=w.T, D=w.D, F=w.F, E=w.E, k=w.k, dtype=w.dtype,
               ms_per_step=ms_per_step, tokens_per_s=w.T / (ms_per_step * 1e-3), step_ms=step_ms,
               working_set_bytes=working_set, precondition_steps=pre_steps, event_pair_overhead_ms=overhead_ms,
               max_expert_share=float(counts.max() / counts.sum()), idle_experts=int((counts == 0).sum()),
               max_expert_rows=int(counts.max()), cold=cold,
               workspace_bytes=layer.workspace_bytes, dominant=dominant, kernels=kernels)
    del layer, inp, y, routing
    torch.cuda.empty_cache()
    return res


def run_static(name, cfs, steps=3, no_drop_rows=0):
    """The static-capacity baseline on the same workload: every expert owns cf * k*T/E rows,
    overflow is dropped, unused rows are zero and still computed.  Both the index-moved and the
    one-hot-mask ("einsum") forms.  no_drop_rows > 0 adds the index-moved form at that capacity -- the
    busiest expert's row count, i.e. the smallest capacity that drops nothing, which is where the paper's
    waste factor (rows computed / rows needed, Sec. 3.2) shows without the drops hiding it."""
    import torch
    from paper_2303_06182_amd import binding, workloads as wl

    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w, device="cuda")
    layer = binding.MoeLayer(w.T, w.D, w.F, w.E, w.k, w.dtype)
    y = torch.empty((w.T, w.D), dtype=w.torch_dtype, device="cuda")
    out = {}
    runs = []
    for cf in cfs:
        cap = binding.moe_capacity(w.T, w.E, w.k, cf, binding.MOE_CAPACITY_SHARE)
        runs.append(("cf%.1f_indexed" % cf, cap, binding.MOE_STATIC_INDEXED))
        runs.append(("cf%.1f_einsum" % cf, cap, binding.MOE_STATIC_EINSUM))
    if no_drop_rows > 0:
        runs.append(("no_drop_indexed", int(no_drop_rows), binding.MOE_STATIC_INDEXED))
    for label, cap, mode in runs:
        nbytes = layer.moe_static_workspace_bytes(w.T, cap, mode)
        free, _ = torch.cuda.mem_get_info()
        if nbytes > free - (8 << 30):
            out[label] = dict(capacity_rows=cap, skipped="workspace of %d bytes does not fit" % nbytes)
            continue
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")

        def step():
            return layer.moe_layer_forward_static(inp["x"], inp["wg"], inp["w1"], inp["w2"], cap, mode,
                                                  inp["gate_bias"], y=y, workspace=ws)
        _, dropped = step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            step()
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / steps
        out[label] = dict(
            capacity_rows=cap, padded_rows=cap * w.E, needed_rows=w.k * w.T, waste_factor=cap * w.E / (w.k * w.T),
            dropped_assignments=int(dropped[0]), ms_per_step=ms, tokens_per_s=w.T / (ms * 1e-3),
            workspace_bytes=nbytes)
        del ws
        torch.cuda.empty_cache()
    del layer, inp, y
    torch.cuda.empty_cache()
    return out


def run_buffering(name, slots_list, n_steps, rho=0.9, tokens=(64, 16)):
    """Expert Buffering (paper Sec. 6) on a decode-shaped workload: the expert parameters stay in
    pinned host memory, `slots` experts fit on the device, a synthetic sequence of decode steps with
    temporally correlated expert activity runs through moe_layer_forward_buffered.  Reports the
    throughput, the cache's miss rate and the copied bytes per cache size, beside the plain call
    (all experts resident).  The observed activity trace is kept for the CPU-baseline leg, which
    simulates the paper's policy, FIFO, LRU and Belady's MIN on it (cpu_cache_policies)."""
    import torch
    from paper_2303_06182_amd import binding, workloads as wl

    base = wl.CONFIGS[name]
    inp = wl.make_inputs(base, device="cpu")
    hw1, hw2 = inp["w1"].pin_memory(), inp["w2"].pin_memory()
    g = {k: (None if v is None else v.cuda()) for k, v in inp.items()}
    results = {}
    for T in tokens:  # the workload as defined, and a sparser step (a quarter of the tokens: about 3/4 of the experts idle)
        results["T%d" % T] = _buffering_runs(base.scaled(T=T), g, hw1, hw2, slots_list, n_steps, rho)
    # the same buffer over quantised expert weights (not in the paper): fewer bytes per missed expert
    del hw1, hw2
    layer = binding.MoeLayer(base.T, base.D, base.F, base.E, base.k, base.dtype)
    for label, wbits, quant in (("e4m3", 8, layer.moe_quantize_e4m3), ("mxfp4", 4, layer.moe_quantize_mxfp4)):
        q1, s1 = quant(g["w1"])
        q2, s2 = quant(g["w2"])
        torch.cuda.synchronize()
        fmt = dict(wbits=wbits, q1=q1, q2=q2, s1=s1, s2=s2)
        hq1, hq2 = q1.cpu().pin_memory(), q2.cpu().pin_memory()
        results["T%d_%s" % (tokens[0], label)] = _buffering_runs(base.scaled(T=tokens[0]), g, hq1, hq2, slots_list,
                                                                 n_steps, rho, fmt)
        del fmt, q1, q2, hq1, hq2
        torch.cuda.empty_cache()
    return results


def _buffering_runs(w, g, hw1, hw2, slots_list, n_steps, rho, fmt=None):
    import numpy as np
    import torch
    from paper_2303_06182_amd import binding, workloads as wl

    name = w.name
    xs = [x.cuda() for x in wl.decode_steps(w, n_steps, rho)]
    layer = binding.MoeLayer(w.T, w.D, w.F, w.E, w.k, w.dtype)
    y = torch.empty((w.T, w.D), dtype=w.torch_dtype, device="cuda")
    routing = layer.empty_routing(w.T)
    wbits = fmt["wbits"] if fmt else 0
    expert_bytes = 2 * w.F * w.D * wbits // 8 if fmt else 2 * w.F * w.D * (2 if w.dtype == "bf16" else 4)

    def resident(x, **kw):
        if not fmt:
            layer.moe_layer_forward(x, g["wg"], g["w1"], g["w2"], g["gate_bias"], y=y, **kw)
        elif wbits == 8:
            layer.moe_layer_forward_w8(x, g["wg"], fmt["q1"], fmt["q2"], fmt["s1"], fmt["s2"], g["gate_bias"], y=y, **kw)
        else:
            layer.moe_layer_forward_w4(x, g["wg"], fmt["q1"], fmt["q2"], fmt["s1"], fmt["s2"], g["gate_bias"], y=y, **kw)

    trace = []
    for x in xs:  # plain call: warm-up and the activity trace
        resident(x, routing_out=routing)
        trace.append(np.nonzero(routing["counts"].cpu().numpy())[0].tolist())
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for x in xs:
        resident(x)
    torch.cuda.synchronize()
    plain_ms = (time.perf_counter() - t0) * 1e3 / n_steps
    out = dict(workload=name, weights="bf16" if not fmt else ("e4m3" if wbits == 8 else "mxfp4"), steps=n_steps, rho=rho,
               expert_bytes=expert_bytes,
               active_experts_per_step=float(np.mean([len(t) for t in trace])),
               distinct_experts=len(set(e for t in trace for e in t)),
               all_resident=dict(ms_per_step=plain_ms, tokens_per_s=w.T / (plain_ms * 1e-3),
                                 expert_bytes_on_device=w.E * expert_bytes),
               slots={}, activity_trace=trace)
    for slots in slots_list:
        cache = (binding.ExpertCache(layer, slots, hw1, hw2, wbits, fmt["s1"], fmt["s2"]) if fmt
                 else binding.ExpertCache(layer, slots, hw1, hw2))
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for x in xs:
            cache.moe_layer_forward_buffered(x, g["wg"], g["gate_bias"], y=y)
        torch.cuda.synchronize()
        secs = time.perf_counter() - t0
        st = cache.stats()
        ms = secs * 1e3 / n_steps
        out["slots"][str(slots)] = dict(
            ms_per_step=ms, tokens_per_s=w.T / (ms * 1e-3), hits=st["hits"], misses=st["misses"],
            miss_rate=st["misses"] / max(1, st["hits"] + st["misses"]), bytes_copied=st["bytes_copied"],
            copy_GBps_over_wall_time=st["bytes_copied"] / secs / 1e9, stages_per_step=st["stages"] / n_steps,
            expert_bytes_on_device=slots * expert_bytes, device_bytes_saved=(w.E - slots) * expert_bytes)
        del cache
        torch.cuda.empty_cache()
    return out


def run_weight_formats(name, steps=20, warmup=4, profile_steps=5):
    """The same workload with the expert weights stored as bf16, as e4m3 bytes (moe_layer_forward_w8)
    and as e2m1 nibbles with block scales (moe_layer_forward_w4): whole-layer time and the two expert
    GEMMs against the HBM roof, the weight bytes counted at their stored size."""
    import numpy as np
    import torch
    from paper_2303_06182_amd import binding, workloads as wl

    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w, device="cuda")
    layer = binding.MoeLayer(w.T, w.D, w.F, w.E, w.k, w.dtype)
    y = torch.empty((w.T, w.D), dtype=w.torch_dtype, device="cuda")
    routing = layer.empty_routing(w.T)
    q1, s1 = layer.moe_quantize_e4m3(inp["w1"])
    q2, s2 = layer.moe_quantize_e4m3(inp["w2"])
    p1, t1 = layer.moe_quantize_mxfp4(inp["w1"])
    p2, t2 = layer.moe_quantize_mxfp4(inp["w2"])
    torch.cuda.synchronize()

    def step16():
        layer.moe_layer_forward(inp["x"], inp["wg"], inp["w1"], inp["w2"], inp["gate_bias"], y=y, routing_out=routing)

    def step8():
        layer.moe_layer_forward_w8(inp["x"], inp["wg"], q1, q2, s1, s2, inp["gate_bias"], y=y, routing_out=routing)

    def step4():
        layer.moe_layer_forward_w4(inp["x"], inp["wg"], p1, p2, t1, t2, inp["gate_bias"], y=y, routing_out=routing)

    out = {}
    # bytes per weight: 4-bit elements plus one scale byte per 32
    for label, step, wbytes in (("bf16", step16, 2.0), ("e4m3", step8, 1.0), ("mxfp4", step4, 0.5 + 1.0 / 32)):
        for _ in range(warmup):
            step()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(steps):
            step()
        torch.cuda.synchronize()
        ms = (time.perf_counter() - t0) * 1e3 / steps
        acc = {}
        for _ in range(profile_steps):
            layer.moe_profile_begin()
            step()
            for kname, kms in layer.moe_profile_end():
                acc.setdefault(kname, []).append(kms)
        counts = routing["counts"].cpu().numpy()
        e_active, N = int((counts > 0).sum()), w.k * w.T
        gemms = {}
        for kname in ("expert_gemm1", "expert_gemm2"):
            kms = float(np.mean(acc[kname]))
            nbytes = int(e_active * w.F * w.D * wbytes) + N * (w.D + w.F) * 2
            gemms[kname] = dict(avg_ms=kms, algorithmic_bytes=nbytes, achieved=nbytes / (kms * 1e-3) / 1e9,
                                unit="GB/s", frac=nbytes / (kms * 1e-3) / 1e9 / HBM_PEAK_GBS)
        out[label] = dict(ms_per_step=ms, tokens_per_s=w.T / (ms * 1e-3), kernels=gemms)
    out["speedup_e4m3"] = out["bf16"]["ms_per_step"] / out["e4m3"]["ms_per_step"]
    out["speedup_mxfp4"] = out["bf16"]["ms_per_step"] / out["mxfp4"]["ms_per_step"]
    out["workload"] = name
    del layer, inp, y, routing, q1, q2, p1, p2
    torch.cuda.empty_cache()
    return out


def yardsticks():
    """What the box itself reaches, measured in the same process: a plain device-to-device copy (HBM
    read + write) and the vendor library's dense bf16 GEMM on the two expert-GEMM shapes of mt_encoder.
    Context for the roofline fractions, which stay quoted against the nominal peaks."""
    import torch
    out = {}
    src = torch.empty(1 << 30, dtype=torch.uint8, device="cuda")
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(20):
        dst.copy_(src)
    torch.cuda.synchronize()
    out["copy_GBps"] = 20 * 2 * (1 << 30) / (time.perf_counter() - t0) / 1e9
    del src, dst
    gemms = {}
    for label, (M, K, N) in (("M32768_K2048_N8192", (32768, 2048, 8192)), ("M32768_K8192_N2048", (32768, 8192, 2048))):
        a = torch.randn(M, K, device="cuda", dtype=torch.bfloat16)
        b = torch.randn(N, K, device="cuda", dtype=torch.bfloat16)
        for _ in range(3):
            torch.matmul(a, b.t())
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(10):
            torch.matmul(a, b.t())
        torch.cuda.synchronize()
        gemms[label] = 10 * 2.0 * M * K * N / (time.perf_counter() - t0) / 1e12
        del a, b
    out["vendor_bf16_gemm_TFLOPs"] = gemms
    torch.cuda.empty_cache()
    return out


def cpu_baseline(name, sample_tokens, seed=12345):
    """The CPU oracle as it stands, timed on the host cores on a bounded sample of the same workload: the
    gate, top-k and routing for EVERY token, the expert FFN and combine for `sample_tokens` tokens (each
    output row depends only on its own token, so a sample is exact).  The sample holds, for every expert
    with rows, the first and the last token routed to it, and is filled up with a seeded random choice."""
    import numpy as np
    import torch
    from oracle import moe_oracle as orc
    from paper_2303_06182_amd import workloads as wl

    w = wl.CONFIGS[name]
    inp = wl.make_inputs(w, device="cuda")
    host = {k: (None if v is None else v.cpu()) for k, v in inp.items()}
    del inp
    torch.cuda.empty_cache()
    n = min(w.T, sample_tokens)
    t0 = time.perf_counter()
    logits = orc.gate_logits(host["x"], host["wg"], host["gate_bias"])
    idx, gw = orc.topk(logits, w.k)
    counts, offsets, dst_row, src_tok = orc.route(idx, w.E)
    t_route = time.perf_counter() - t0
    must = set()
    for e in range(w.E):
        if counts[e] > 0:
            must.add(int(src_tok[offsets[e]]))
            must.add(int(src_tok[offsets[e + 1] - 1]))
    rest = [int(t) for t in np.random.default_rng(seed).permutation(w.T) if int(t) not in must]
    tokens = np.array(sorted(must) + rest[:max(0, n - len(must))], dtype=np.int32)
    t0 = time.perf_counter()
    orc.layer_tokens(host["x"], host["w1"], host["w2"], idx, gw, tokens=tokens)
    t_ffn = time.perf_counter() - t0
    per_token = t_route / w.T + t_ffn / len(tokens)
    experts_hit = len(set(idx[tokens].ravel().tolist()))
    return dict(value=1.0 / per_token, unit="tokens/s", cores=orc.n_threads(), kind="oracle",
                sample="workload %s: gate + top-k + routing of all %d tokens (%.2f s) + expert FFN and combine of "
                       "%d tokens (%.2f s; seeded sample with every active expert's first and last token: %d of %d "
                       "active experts hit), tokens/s = 1 / (routing s per token + FFN s per token)"
                       % (name, w.T, t_route, len(tokens), t_ffn, experts_hit, int((counts > 0).sum())))


def cpu_cache_policies(buffering):
    """Part of the CPU-baseline leg: the oracle's cache simulator (paper policy, FIFO, LRU, Belady's MIN;
    Sec. 6) on the expert-activity traces the expert-buffering runs observed."""
    from oracle import expert_cache as ec
    for run in buffering.values():
        trace = run.get("activity_trace")
        if trace is None:
            continue
        run["simulated_miss_rate"] = {slots: {pol: ec.simulate(trace, int(slots), pol)["miss_rate"]
                                              for pol in ec.POLICIES} for slots in run["slots"]}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--config", default="skewed_large", help="headline workload (default: the largest, skewed_large)")
    ap.add_argument("--also", default="lm,mt_encoder,mt_decoder,tiny_f32",
                    help="comma list of further workloads reported under 'also' (the static baseline runs only "
                         "for the headline workload and lm)")
    ap.add_argument("--cpu-tokens", type=int, default=16384,
                    help="tokens of the CPU oracle's FFN sample (0 = skip the whole CPU-baseline leg)")
    ap.add_argument("--no-static", action="store_true", help="skip the static-capacity baseline runs")
    ap.add_argument("--no-buffering", action="store_true", help="skip the expert-buffering runs")
    ap.add_argument("--no-w8", action="store_true", help="skip the run with 8- and 4-bit expert weights (mt_decoder)")
    ap.add_argument("--no-yardsticks", action="store_true", help="skip the box's own copy bandwidth and vendor GEMM rate")
    ap.add_argument("--buffering-steps", type=int, default=16, help="decode steps of the expert-buffering runs")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="first run a plain 1 GiB read + 1 GiB write elementwise kernel three times (untimed): gives counter runs "
                         "(rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE) a kernel of known traffic to scale by")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU (no collectives, no sharding); --gpus %d is not supported"
              % args.gpus, file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2303_06182_amd import binding, workloads as wl
    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    binding.load_library()

    if args.copy_calibration:
        # an int32 "+1" over 1 GiB: reads 1 GiB, writes 1 GiB, in a kernel no other step of this run uses
        src = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.add(src, 1, out=dst)
        torch.cuda.synchronize()
        del src, dst
        torch.cuda.empty_cache()

    def cold_copies_for(name):
        # enough copies of the weights to overflow the last-level cache twice, when one copy fits it
        w = wl.CONFIGS[name]
        wbytes = 2 * w.E * w.D * w.F * (2 if w.dtype == "bf16" else 4)
        return 0 if wbytes > LAST_LEVEL_CACHE_BYTES else int(2 * LAST_LEVEL_CACHE_BYTES // wbytes) + 1

    main_res = run_config(args.config, args.steps, args.warmup, cold_copies=cold_copies_for(args.config))
    also = {}
    max_rows = {args.config: main_res["max_expert_rows"]}
    for name in [a for a in args.also.split(",") if a and a != args.config]:
        r = run_config(name, args.steps, args.warmup, profile_steps=5, cold_copies=cold_copies_for(name))
        max_rows[name] = r["max_expert_rows"]
        also[name] = dict(tokens_per_s=r["tokens_per_s"], ms_per_step=r["ms_per_step"], step_ms=r["step_ms"],
                          working_set_bytes=r["working_set_bytes"], roofline=r["dominant"], cold=r["cold"],
                          kernels={k: dict(avg_ms=v["avg_ms"], bound=v["bound"], frac=v["frac"], traffic=v["traffic"])
                                   for k, v in r["kernels"].items()},
                          max_expert_share=r["max_expert_share"])
    static = {}
    if not args.no_static:
        for name in [args.config] + [n for n in also if n == "lm"]:
            static[name] = run_static(name, [1.0, 2.0], no_drop_rows=max_rows[name])
    buffering = None
    if not args.no_buffering:
        buffering = run_buffering("mt_decoder", [16, 48, 96], args.buffering_steps)
    w8 = None if args.no_w8 else run_weight_formats("mt_decoder")
    yard = None if args.no_yardsticks else yardsticks()
    cpu = None
    if args.cpu_tokens > 0:  # the CPU-baseline leg: the only part of this script that touches oracle/
        cpu = cpu_baseline(args.config, args.cpu_tokens)
        if buffering:
            cpu_cache_policies(buffering)
    for run in (buffering or {}).values():
        run.pop("activity_trace", None)

    dom = dict(main_res["dominant"])
    out = {
        "metric": "MoE-layer tokens/s (dynamic gating)",
        "value": main_res["tokens_per_s"],
        "unit": "tokens/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": main_res["ms_per_step"],
        "step_ms": main_res["step_ms"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": main_res["dtype"],
        "data": "synthetic",
        "config": {"workload": args.config, "T": main_res["T"], "D": main_res["D"], "F": main_res["F"],
                   "E": main_res["E"], "k": main_res["k"], "max_expert_share": main_res["max_expert_share"],
                   "idle_experts": main_res["idle_experts"], "workspace_bytes": main_res["workspace_bytes"],
                   "working_set_bytes": main_res["working_set_bytes"],
                   "precondition_seconds": PRECONDITION_SECONDS, "precondition_steps": main_res["precondition_steps"]},
        "roofline": {k: dom[k] for k in ("bound", "achieved", "peak", "unit", "frac", "traffic", "kernel", "avg_ms",
                                                "algorithmic_bytes", "algorithmic_flops")},
        "cpu_baseline": cpu,
        "kernels": {k: dict(avg_ms=v["avg_ms"], event_ms=v["event_ms"], bound=v["bound"], achieved=v["achieved"],
                            unit=v["unit"], frac=v["frac"], traffic=v["traffic"],
                            **({"in_fused_call": False} if not v.get("in_fused_call", True) else {}))
                    for k, v in main_res["kernels"].items()},
        "event_pair_overhead_ms": main_res["event_pair_overhead_ms"],
        "cold": main_res["cold"],
        "also": also,
        "static_baseline": static,
        "expert_buffering": buffering,
        "weight_formats": w8,
        "yardsticks": yard,
        "paper_context": "paper reports only relative whole-model speedups of dynamic over static gating on "
                         "8xV100 nodes (LM 6.21-11.23x, MT encoder 5.75-10.98x, MT decoder 2.58-5.71x); "
                         "no absolute number exists for this metric",
    }
    print(json.dumps(out))


if __name__ == "__main__":
    main()
