"""Benchmark of the pair-search hot path on one MI355X.

One step = one sop_pair_search call over one synthetic layer (block statistics, scale encode,
nearest-entry search for every atom, block scores, selector bits of every pair, layer reduction),
with weights, channel norms and codebook tables already resident in HBM.  The codebook tables are
built and uploaded once per alphabet before the timed region (they do not depend on the layer).

Workload: the headline configuration -- MLP down-projection 4096 x 11008, bf16 Student-t(4)
weights, log-normal channel norms, g = 16, UE4M4 block scale, atoms NF4 / SH4 / BOF4 and their sign
negations, all 15 pairs, selector bits and per-atom / per-pair ACos out.  The layer rotates through
several distinct weight buffers so consecutive steps cannot be served from the 256 MB last-level
cache.

Prints one JSON line.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

CLOCK_RAMP_MS = 60.0            # untimed repetition of the call before the timed region (GPU clock ramp)
HBM_PEAK_GBS = 8000.0           # MI355X HBM3E, published
# Plain vector-ALU peak: the published fp32 vector rate, 157.3 TFLOP/s, counts an fma as two: 78.6e12 fp32
# lane-operations per second with an fma counted once = 256 CUs x 4 SIMDs x 32 lanes per clock x 2.4 GHz.  A SIMD takes
# plain two-operand arithmetic on vector registers (fma, multiply, add, logic, integer add) from two wavefronts at a
# time (measured: 70e12 with four or more wavefronts per SIMD, 2.3 cycles an instruction; 2.8 cycles with three,
# where one wavefront goes alone; `--workload issue_probe`); compares, selects, minima and maxima, conversions, left
# shifts, three-operand integer forms and anything with a scalar-register operand are taken at half that rate
# (VALU_HALF_RATE_TLOPS) but leave the other slot to the first class, so a mixed stream runs at the first rate.
# Packed fp32 (two operations per lane) is not used in this build.
VALU_PEAK_TLOPS = 78.6432
VALU_HALF_RATE_TLOPS = 39.3216


def algorithmic_lane_ops(n_weights, g, n_atoms, n_groups, n_pairs, signs=1, n_copies=0):
    """Lane-operations of the method's own arithmetic per launch (an fma counted once), not of the code:
    per weight: widen, max, min, c*w, ||w||^2 fma                                    = 5
    per weight and scale group: x = w*r, the two operations that locate x's code     = 3
    per weight and evaluated (atom, sign): compare with the code boundary, select
        the entry, residual fma, c*d, error fma, cosine-sum fma                      = 6
        (the kernel spends a seventh, forming the boundary from the table's two values: not the method's)
    per block and scale group: ideal scale 3, shift 1, encode 5, decode+reciprocal 3 = 12
    per block and atom: chunk add 1, cosine 5, accumulate 2                          = 8
    per block and pair: compare, select, add, two operations for the selector bit    = 5
    A signed scale word evaluates both signs of every atom (groups and atoms count twice, three more
    operations per block and atom keep the better sign), except that an atom that is the sign-negated copy
    of another (n_copies of the n_atoms) takes its candidates over from it and is not evaluated."""
    evaluated = n_atoms - (n_copies if signs == 2 else 0)
    per_weight = 5 + signs * (3 * n_groups + 6 * evaluated)
    per_block = signs * 12 * n_groups + 8 * n_atoms + (signs - 1) * (8 * evaluated + 3 * n_atoms) + 5 * n_pairs
    return n_weights * per_weight + (n_weights // g) * per_block


def parse_traffic():
    """Measured HBM bytes per launch from the committed rocprofv3 counter summary, when present."""
    path = os.path.join(ROOT, "profiles", "search_kernel_c3down_hbm_traffic.txt")
    if not os.path.exists(path):
        return None
    vals = {}
    for line in open(path):
        line = line.split("#", 1)[0]
        if "=" in line:
            k, v = line.split("=", 1)
            try:
                vals[k.strip()] = float(v)
            except ValueError:
                pass
    if "hbm_bytes_per_launch" in vals:
        return vals["hbm_bytes_per_launch"]
    return None


def counters_from_file():
    """Figures of the headline kernel that this run does NOT measure: they are read from the committed rocprofv3
    counter summary (profiles/search_kernel_c3down_valu.txt, taken with `rocprofv3 --pmc` on this workload) and
    are labelled as such in the bench line."""
    path = os.path.join(ROOT, "profiles", "search_kernel_c3down_valu.txt")
    if not os.path.exists(path):
        return None
    vals = {}
    for line in open(path):
        line = line.split("#", 1)[0]
        if "=" in line:
            k, v = line.split("=", 1)
            try:
                vals[k.strip()] = float(v)
            except ValueError:
                pass
    if "SQ_INSTS_VALU" not in vals:
        return None
    out = {"from_file": "profiles/search_kernel_c3down_valu.txt", "measured_in_this_run": False,
           "wave_valu_instructions_per_launch": vals["SQ_INSTS_VALU"]}
    if "weights_per_launch" in vals:
        out["executed_lane_ops_per_weight"] = vals["SQ_INSTS_VALU"] * 64.0 / vals["weights_per_launch"]
    return out


def timed_region(step, steps):
    """K calls back to back between one HIP event before and one after on the launch stream (events
    inside the loop would put a marker between every two kernels).  Returns (wall ms per step, GPU ms
    per step)."""
    import torch
    # The GPU raises its clock over the first 20-30 ms of load.  Whatever --warmup says, the same call is
    # repeated untimed for CLOCK_RAMP_MS first, so that a short run is not timed inside that ramp.
    t_ramp = time.perf_counter()
    j = 0
    while (time.perf_counter() - t_ramp) * 1e3 < CLOCK_RAMP_MS:
        for _ in range(20):
            step(j)
            j += 1
        torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record()
    for i in range(steps):
        step(i)
    e1.record()
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) / steps * 1e3, e0.elapsed_time(e1) / steps


def bench_probe(args):
    """Calibration: a plain read of the headline layer's bytes (and of the 70B-shaped layer's) by the
    library's read-probe kernel; the time is the floor of every pass that reads a layer once."""
    import torch
    import paper_2605_14929_amd as sop
    dev = torch.device("cuda", 0)
    ctx = sop.Context(0)
    out = torch.empty(2048, dtype=torch.int32, device=dev)
    res = {}
    for label, M, K, n_buf in (("4096x11008 bf16", 4096, 11008, args.buffers), ("28672x8192 bf16", 28672, 8192, 3)):
        bufs = [torch.randint(-(1 << 31), (1 << 31) - 1, (M * K // 2,), dtype=torch.int32, device=dev) for _ in range(n_buf)]
        for i in range(args.warmup):
            ctx.read_probe(bufs[i % n_buf], out)
        torch.cuda.synchronize()
        ms_step, ev_ms = timed_region(lambda i: ctx.read_probe(bufs[i % n_buf], out), args.steps)
        nbytes = M * K * 2
        res[label] = {"bytes": nbytes, "event_ms_per_launch": ev_ms, "GB/s": nbytes / (ev_ms * 1e-3) / 1e9,
                      "frac_of_published_peak": nbytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "buffers_rotated": n_buf}
        del bufs
    head = res["4096x11008 bf16"]
    result = {
        "metric": "bytes read/sec (plain read, calibration)", "value": head["GB/s"] * 1e9, "unit": "B/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": head["event_ms_per_launch"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": "plain read of 90 MB (the C3 down-projection's bytes) by sopk::read_probe_kernel"},
        "roofline": {"bound": "hbm", "achieved": head["GB/s"], "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": head["frac_of_published_peak"],
                     "traffic": None, "algorithmic_bytes_per_launch": head["bytes"], "kernel": "sopk::read_probe_kernel",
                     "event_ms_per_launch": head["event_ms_per_launch"]},
        "sizes": res, "untimed_clock_ramp_ms": CLOCK_RAMP_MS,
    }
    print(json.dumps(result))


def bench_issue(args):
    """Calibration: the rate at which the vector ALUs take instructions of one kind, by the number of wavefronts
    a SIMD holds (the library's issue-probe kernel: no memory traffic, eight independent chains per lane)."""
    import torch
    import paper_2605_14929_amd as sop
    dev = torch.device("cuda", 0)
    ctx = sop.Context(0)
    n_cu = torch.cuda.get_device_properties(dev).multi_processor_count
    kinds = ["v_fmac_f32 (registers only)", "v_max_f32", "v_fma_f32 with a scalar-register operand", "v_cmp_lt_f32 + v_cndmask_b32",
             "v_mul_f32", "v_mad_u32_u24", "v_fma_f32 + v_max_f32 alternating", "v_add_f32", "v_and_b32", "v_add_u32", "v_lshrrev_b32",
             "v_lshlrev_b32", "v_cvt_i32_f32", "v_med3_f32", "v_rcp_f32",
             "element pass, 12-byte look-ups (6 instructions per element)", "element pass, 8-byte look-ups (7 instructions per element)",
             "element pass, no look-ups (7 instructions per element)", "element pass, no look-ups (6 instructions per element)"]
    per_iter = {15: 96 * 6, 16: 96 * 7, 17: 96 * 7, 18: 96 * 6}          # vector instructions per lane and iteration (the other kinds: 64)
    out = torch.empty(n_cu * 8 * 256, dtype=torch.float32, device=dev)
    table = {}
    for kind, name in enumerate(kinds):
        row = {}
        iters = 4000 if kind < 15 else 400
        for wps in ((1, 2, 3, 4, 6, 8) if kind < 7 else ((1, 2, 3, 4) if kind >= 15 else (8,))):     # kinds 7..14: the class only
            for _ in range(3):
                ctx.issue_probe(kind, wps, iters, 1.0, 0.125, out)
            torch.cuda.synchronize()
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            reps = 5
            for _ in range(reps):
                ctx.issue_probe(kind, wps, iters, 1.0, 0.125, out)
            e1.record()
            torch.cuda.synchronize()
            ms = e0.elapsed_time(e1) / reps
            wave_instr = n_cu * 4 * wps * iters * float(per_iter.get(kind, 64))
            row[str(wps)] = {"ms": ms, "T_lane_ops_per_s": wave_instr * 64 / (ms * 1e-3) / 1e12,
                             "cycles_per_instruction_per_simd_at_2.4GHz": ms * 1e-3 * 2.4e9 * n_cu * 4 / wave_instr}
            if kind >= 15:      # SIMD cycles per element of a pass (per weight and codebook in the search kernel)
                row[str(wps)]["cycles_per_element_per_simd_at_2.4GHz"] = ms * 1e-3 * 2.4e9 * n_cu * 4 / (n_cu * 4 * wps * iters * 96.0)
        table[name] = row
    best = table[kinds[0]]["8"]["T_lane_ops_per_s"]
    result = {
        "metric": "vector-ALU lane-operations/sec (issue-rate calibration)", "value": best * 1e12, "unit": "lane-ops/s", "n_gpus": 1,
        "steps": 5, "warmup": 3, "ms_per_step": table[kinds[0]]["8"]["ms"], "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "sopk::issue_probe_kernel: 64 instructions of one kind per lane and iteration, by kind and by wavefronts per SIMD"},
        "roofline": {"bound": "alu", "achieved": best, "peak": VALU_PEAK_TLOPS, "unit": "T lane-ops/s", "frac": best / VALU_PEAK_TLOPS,
                     "traffic": None, "kernel": "sopk::issue_probe_kernel<0>"},
        "by_kind_and_wavefronts_per_simd": table,
    }
    print(json.dumps(result))


def bench_dd(args):
    """Statistics pass of the data-derived codebook on the headline layer (whole layer, 4096 bins):
    every weight is read once and adds its channel norm to one histogram bin."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si
    W, c, cfg = si.make_config("C3_down")
    M, K, g, H = cfg["M"], cfg["K"], cfg["g"], 4096
    dev = torch.device("cuda", 0)
    w0 = torch.from_numpy(W).to(dev).to(torch.bfloat16)
    bufs = [w0] + [torch.roll(w0, shifts=17 * i, dims=0).contiguous() for i in range(1, args.buffers)]
    ct = torch.from_numpy(c).to(dev)
    ctx = sop.Context(0)
    for i in range(args.warmup):
        ctx.dd_histogram(bufs[i % len(bufs)], ct, g, H)
    torch.cuda.synchronize()
    ms_step, ev_ms = timed_region(lambda i: ctx.dd_histogram(bufs[i % len(bufs)], ct, g, H), args.steps)
    alg_bytes = M * K * 2 + K * 4 + H * 8
    result = {
        "metric": "weights histogrammed/sec", "value": M * K / (ms_step * 1e-3), "unit": "weights/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "int64", "data": "synthetic",
        "config": {"workload": "DD histogram of the C3 down-projection 4096x11008 bf16, g=16, 4096 bins, channel-norm weights, every row",
                   "M": M, "K": K, "g": g, "n_bins": H},
        "layer_latency_ms": ev_ms,
        "roofline": {"bound": "hbm", "achieved": alg_bytes / (ev_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": alg_bytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "traffic": None,
                     "algorithmic_bytes_per_launch": alg_bytes, "kernel": "sopk::dd_hist_kernel", "event_ms_per_launch": ev_ms,
                     "note": "the pass is held back by LDS atomic throughput (one LDS atomic per weight), not by HBM"},
    }
    if not args.no_cpu_baseline:
        from oracle import dd as DD
        rows = M
        t0 = time.perf_counter()
        ref = DD.histogram(W[:rows], c, g, H)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": rows * K / dt, "unit": "weights/s", "cores": 1, "kind": "oracle",
                                  "sample": f"the whole layer ({rows} rows), numpy on one core, {dt:.2f} s wall"}
        chk = ctx.dd_histogram(torch.from_numpy(W[:rows]).to(dev).to(torch.bfloat16), ct, g, H)
        torch.cuda.synchronize()
        result["parity_in_run"] = {"histogram_equal": bool(np.array_equal(chk.cpu().numpy(), ref))}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def bench_fl(args):
    """Statistics pass of the per-layer scale shift on the headline layer: every weight is read once,
    one counter update per block."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si
    W, c, cfg = si.make_config("C3_down")
    M, K, g = cfg["M"], cfg["K"], cfg["g"]
    fmt = sop.fmt_by_name(cfg["fmt"])
    dev = torch.device("cuda", 0)
    w0 = torch.from_numpy(W).to(dev).to(torch.bfloat16)
    bufs = [w0] + [torch.roll(w0, shifts=17 * i, dims=0).contiguous() for i in range(1, args.buffers)]
    ctx = sop.Context(0)
    for i in range(args.warmup):
        ctx.scale_histogram(bufs[i % len(bufs)], g, 1.0, 1.0, fmt)
    torch.cuda.synchronize()
    ms_step, ev_ms = timed_region(lambda i: ctx.scale_histogram(bufs[i % len(bufs)], g, 1.0, 1.0, fmt), args.steps)
    alg_bytes = M * K * 2 + 640 * 8
    result = {
        "metric": "blocks scanned/sec", "value": M * K // g / (ms_step * 1e-3), "unit": "blocks/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "block-scale exponent histogram of the C3 down-projection 4096x11008 bf16, g=16, UE4M4, unit endpoints",
                   "M": M, "K": K, "g": g},
        "layer_latency_ms": ev_ms,
        "roofline": {"bound": "hbm", "achieved": alg_bytes / (ev_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": alg_bytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "traffic": None,
                     "algorithmic_bytes_per_launch": alg_bytes, "kernel": "sopk::scale_hist_kernel", "event_ms_per_launch": ev_ms},
    }
    if not args.no_cpu_baseline:
        from oracle import flayer as FL
        t0 = time.perf_counter()
        sc = FL.block_scales(W, g, 1.0, 1.0)
        ref = FL.exponent_histogram(sc, fmt.exp_bits, fmt.man_bits, fmt.bias, fmt.max_code)
        k_ref = FL.layer_shift(sc, fmt.exp_bits, fmt.man_bits, fmt.bias, fmt.max_code)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": M * K // g / dt, "unit": "blocks/s", "cores": 1, "kind": "oracle",
                                  "sample": f"the whole layer, numpy on one core (scales, histogram and the search over k), {dt:.2f} s wall"}
        chk = ctx.scale_histogram(bufs[0], g, 1.0, 1.0, fmt)
        torch.cuda.synchronize()
        h = chk.cpu().numpy()
        result["parity_in_run"] = {"histogram_equal": bool(np.array_equal(h, ref)),
                                   "k_star": sop.sop_layer_shift(h, M * K // g, fmt)[0], "k_star_oracle": k_ref[0]}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def bench_ls(args):
    """Layer-scope FP8 baseline (E4M3 weights, one power-of-two scale per layer) on the headline layer:
    one pass for the layer maxima, one pass rounding every weight and summing the errors."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si
    W, c, cfg = si.make_config("C3_down")
    M, K = cfg["M"], cfg["K"]
    wf, sf = sop.WeightFmt(4, 3, -1, -1), sop.ScaleFmt(0, 8, 0, 8, 127, 252)
    dev = torch.device("cuda", 0)
    w0 = torch.from_numpy(W).to(dev).to(torch.bfloat16)
    bufs = [w0] + [torch.roll(w0, shifts=17 * i, dims=0).contiguous() for i in range(1, args.buffers)]
    ct = torch.from_numpy(c).to(dev)
    ctx = sop.Context(0)
    for i in range(args.warmup):
        ctx.layer_scope_error(bufs[i % len(bufs)], ct, wf, sf)
    torch.cuda.synchronize()
    ms_step, ev_ms = timed_region(lambda i: ctx.layer_scope_error(bufs[i % len(bufs)], ct, wf, sf), args.steps)
    alg_bytes = 2 * (M * K * 2) + K * 4 + 32                        # the layer is read twice: maxima, then rounding
    result = {
        "metric": "weights rounded/sec", "value": M * K / (ms_step * 1e-3), "unit": "weights/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "E4M3^0sUE8M0 reconstruction error of the C3 down-projection 4096x11008 bf16 (layer maxima pass + rounding pass)",
                   "M": M, "K": K},
        "layer_latency_ms": ev_ms,
        "roofline": {"bound": "hbm", "achieved": alg_bytes / (ev_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": alg_bytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "traffic": None,
                     "algorithmic_bytes_per_launch": alg_bytes, "kernel": "sopk::layer_max_kernel + sopk::layer_scope_kernel",
                     "event_ms_per_launch": ev_ms},
    }
    if not args.no_cpu_baseline:
        from oracle import layerscope as LS, pairsearch as ops
        t0 = time.perf_counter()
        ref = LS.layer_scope(W, c, LS.exmy_table(4, 3), ops.make_fmt(0, 8, 0, 8, 127, 252))
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": M * K / dt, "unit": "weights/s", "cores": 1, "kind": "oracle",
                                  "sample": f"the whole layer, numpy on one core, {dt:.2f} s wall"}
        chk, _ = ctx.layer_scope_error(bufs[0], ct, wf, sf)
        torch.cuda.synchronize()
        o = chk.cpu().numpy()
        result["parity_in_run"] = {"scale_code_equal": int(o[3]) == ref["q"], "rel_err_weighted_error": abs(o[0] - ref["err_w"]) / ref["err_w"]}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def bench_finish(args):
    """Steps 2 and 3 of the pair search and the materialisation on the headline layer, after an
    emitting search over (NF4, SH4) with a UE4M3 scale word (one metabit): rank the blocks by their
    cosine under NF4 and split the pools (70% stay), histogram of the fitting pool, pack scale words
    and code payloads of the pair."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si
    W, c, cfg = si.make_config("C3_down")
    M, K, g = cfg["M"], cfg["K"], cfg["g"]
    Nb = M * K // g
    fmt = sop.fmt_by_name("UE4M3")
    tabs = sop.build_alphabet(["NF4", "SH4"])
    dev = torch.device("cuda", 0)
    wt = torch.from_numpy(W).to(dev).to(torch.bfloat16)
    ct = torch.from_numpy(c).to(dev)
    ctx = sop.Context(0)
    ctx.set_alphabet(tabs)
    out = ctx.pair_search(wt, ct, g, fmt, emit=True)
    torch.cuda.synchronize()
    n_top = int(np.floor(0.70 * Nb + 0.5))
    score = out.blk_cos[0]

    def step():
        pool_b, tau, n_a = ctx.partition(score, n_top, True)
        hist = ctx.dd_histogram(wt, ct, g, 1024, 1, block_mask=pool_b)
        words, payload, n = ctx.pack_blocks(out, M, K, g, fmt, 0, 1, 0)
        return pool_b, tau, n_a, hist, words, payload

    for _ in range(args.warmup):
        step()
    ms_step, ev_step_ms = timed_region(lambda i: step(), args.steps)
    # per-part latency with events on the launch stream
    parts = {}
    for name, fn in (("partition", lambda: ctx.partition(score, n_top, True)),
                     ("masked_histogram", lambda: ctx.dd_histogram(wt, ct, g, 1024, 1, block_mask=step.pool)),
                     ("pack", lambda: ctx.pack_blocks(out, M, K, g, fmt, 0, 1, 0))):
        if name == "masked_histogram":
            step.pool = ctx.partition(score, n_top, True)[0]
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(50)]
        for a, b in ev:
            a.record(); fn(); b.record()
        torch.cuda.synchronize()
        parts[name] = float(np.mean([a.elapsed_time(b) for a, b in ev]))
    alg = {"partition": 4 * 4 * Nb + Nb + 12,                         # the score plane is read by each of the four kernels
           "masked_histogram": M * K * 2 + Nb + K * 4 + 8 * 1024,
           "pack": Nb * (2 + 2 + g // 2) + Nb * (2 + g // 2)}
    ev_ms = ev_step_ms                                                  # the whole chain, timed region
    alg_bytes = sum(alg.values())
    result = {
        "metric": "blocks finished/sec", "value": Nb / (ms_step * 1e-3), "unit": "blocks/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "u32", "data": "synthetic",
        "config": {"workload": "steps 2-3 and packing after a (NF4, SH4) UE4M3 search of the C3 down-projection 4096x11008 bf16: "
                               "rank 2.8 M block cosines, 70/30 pools, masked 1024-bin histogram, scale words + 8-byte payloads",
                   "M": M, "K": K, "g": g, "n_top": n_top},
        "part_latency_ms": parts,
        "roofline": {"bound": "hbm", "achieved": alg_bytes / (ev_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": alg_bytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "traffic": None,
                     "algorithmic_bytes_per_launch": alg_bytes, "algorithmic_bytes_by_part": alg,
                     "kernel": "sopk::rank_count_kernel x3 + sopk::rank_split_kernel + sopk::dd_hist_kernel + sopk::pack_kernel",
                     "event_ms_per_launch": ev_ms},
    }
    if not args.no_cpu_baseline:
        from oracle import dd as DD, pack as PK, partition as PT, pairsearch as ops
        Ms = 512                                                       # bounded sample: the first 512 rows
        Ws = W[:Ms]
        ref = ops.pair_search(Ws, c, tabs, g, ops.make_fmt(0, 4, 3))
        t0 = time.perf_counter()
        nbs = Ms * K // g
        rt, rp, rn = PT.partition(ref.blk_cos[0], int(np.floor(0.70 * nbs + 0.5)), True)
        rh = DD.histogram(Ws, c, g, 1024, block_mask=rp)
        rw, rpl, _ = PK.materialise(ref, tabs, Ms, K, g, 0, 1, 0, 0, 4, 3, 8)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": nbs / dt, "unit": "blocks/s", "cores": 1, "kind": "oracle",
                                  "sample": f"the first {Ms} rows of the layer ({nbs} blocks), numpy on one core, {dt:.2f} s wall"}
        # parity in the run: the same rows through the library
        o2 = ctx.pair_search(wt[:Ms], ct, g, fmt, emit=True)
        pb, tau, n_a = ctx.partition(o2.blk_cos[0], int(np.floor(0.70 * nbs + 0.5)), True)
        words, payload, _ = ctx.pack_blocks(o2, Ms, K, g, fmt, 0, 1, 0)
        torch.cuda.synchronize()
        gt, gp, gn = PT.partition(o2.blk_cos[0].cpu().numpy(), int(np.floor(0.70 * nbs + 0.5)), True)
        result["parity_in_run"] = {"words_equal": bool(np.array_equal(words.cpu().numpy().view(np.uint16), rw)),
                                   "payload_equal": bool(np.array_equal(payload.cpu().numpy(), rpl)),
                                   "pool_equal_on_gpu_scores": bool(np.array_equal(pb.cpu().numpy(), gp) and int(n_a.item()) == gn)}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def bench_model(args):
    """Configuration 4: the pair search over all 224 linear layers of a 7B-shaped model (32 blocks of
    q/k/v/o 4096x4096, gate/up 11008x4096, down 4096x11008; bf16, g = 16, UE4M4, six atoms, 15 pairs),
    every layer resident in HBM in its own buffer (13 GB), one call, a [224, 15] ACos table out.
    Block 0 is drawn from the seeded generator (per-layer tail index from U(3,8)); the other 31 blocks
    are row-rotated copies of it made on the GPU (drawing 6.5 G Student-t samples on the host would take
    minutes), each layer with its own channel norms."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si
    n_blocks, g = 32, 16
    tabs = sop.build_alphabet(["NF4", "SH4", "BOF4", "-NF4", "-SH4", "-BOF4"], bof_draws=si.normal_draws(1 << 20, 4242))
    fmt = sop.fmt_by_name("UE4M4")
    dev = torch.device("cuda", 0)
    host = list(si.model_7b_layers(1))
    base = [torch.from_numpy(W).to(dev).to(torch.bfloat16) for _, W, _, _ in host]
    layers = []
    for b in range(n_blocks):
        for i, (_, _, c, _) in enumerate(host):
            Wt = base[i] if b == 0 else torch.roll(base[i], shifts=37 * b, dims=0).contiguous()
            ct = torch.from_numpy(c if b == 0 else si.channel_norms(c.size, 1.0, 900000 + 10 * b + i)).to(dev)
            layers.append((Wt, ct))
    n_weights = sum(W.numel() for W, _ in layers)
    ctx = sop.Context(0)
    ctx.set_alphabet(tabs)
    steps = min(args.steps, 10)
    for _ in range(min(args.warmup, 2)):
        ctx.pair_search_layers(layers, g, fmt)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record()
    for _ in range(steps):
        tp, ta, _ = ctx.pair_search_layers(layers, g, fmt)
    e1.record()
    torch.cuda.synchronize()
    ms_step = (time.perf_counter() - t0) / steps * 1e3
    ev_ms = e0.elapsed_time(e1) / steps
    A, P = 6, 15
    lane_ops = sum(algorithmic_lane_ops(W.numel(), g, A, 3, P) for W, _ in layers)
    alg_bytes = sum(W.numel() * 2 + W.shape[1] * 4 for W, _ in layers) + len(layers) * (A + P) * 8
    result = {
        "metric": "block x atom evaluations/sec", "value": n_weights // g * A / (ms_step * 1e-3), "unit": "block*atom evals/s",
        "n_gpus": 1, "steps": steps, "warmup": min(args.warmup, 2), "ms_per_step": ms_step, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "7B-shaped model, 224 linear layers bf16 (6.48 G weights, 13 GB resident), g=16, UE4M4, 6 atoms, "
                               "15 pairs, ACos table only; one step = the whole model",
                   "layers": len(layers), "weights": n_weights, "distinct_layers_drawn": len(host)},
        "layers_per_second": len(layers) / (ms_step * 1e-3), "model_latency_ms": ev_ms,
        "roofline": {"bound": "alu", "achieved": lane_ops / (ev_ms * 1e-3) / 1e12, "peak": VALU_PEAK_TLOPS, "unit": "T lane-ops/s",
                     "frac": lane_ops / (ev_ms * 1e-3) / 1e12 / VALU_PEAK_TLOPS, "traffic": None,
                     "algorithmic_lane_ops_per_launch": lane_ops, "kernel": "sopk::search_kernel (model-wide variant: one launch for the 224 layers)", "event_ms_per_launch": ev_ms},
        "roofline_hbm": {"bound": "hbm", "achieved": alg_bytes / (ev_ms * 1e-3) / 1e9, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                         "frac": alg_bytes / (ev_ms * 1e-3) / 1e9 / HBM_PEAK_GBS, "algorithmic_bytes_per_launch": alg_bytes},
    }
    if not args.no_cpu_baseline:
        from oracle import atoms as OA, pairsearch as ops
        name, W, c, _ = host[0]                                        # the q projection, whole layer
        otabs = [np.asarray(t, dtype=np.float32) for t in tabs]
        t0 = time.perf_counter()
        ref = ops.pair_search(W, c, otabs, g, ops.make_fmt(0, 4, 4), want_codes=False)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": W.size // g * A / dt, "unit": "block*atom evals/s", "cores": ops.num_threads(), "kind": "oracle",
                                  "sample": f"layer {name} (4096x4096) of the 224, whole layer, {dt:.2f} s wall"}
        result["parity_in_run"] = {"layer": name, "max_abs_dacos_pair": float(np.max(np.abs(tp[0].cpu().numpy() - ref.acos_pair))),
                                   "max_abs_dacos_atom": float(np.max(np.abs(ta[0].cpu().numpy() - ref.acos_atom)))}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def bench_layer_search(args):
    """The whole per-layer procedure on the headline layer: all 15 pairs of the six fixed atoms, then for
    every atom a sweep over p = 50, 70, 85, 95 % with a second codebook fitted on the blocks the atom serves
    worst (24 rankings, 24 masked histograms and fits, 6 scoring calls), the winner packed."""
    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    from paper_2605_14929_amd import layer_search as LSR
    import sop_inputs as si
    W, c, cfg = si.make_config("C3_down")
    M, K, g = cfg["M"], cfg["K"], cfg["g"]
    tabs = sop.build_alphabet(cfg["atoms"], bof_draws=si.normal_draws(1 << 20, 4242))
    fmt = sop.fmt_by_name("UE4M3")                                     # one metabit for the selector
    dev = torch.device("cuda", 0)
    wt = torch.from_numpy(W).to(dev).to(torch.bfloat16)
    ct = torch.from_numpy(c).to(dev)
    ctx = sop.Context(0)
    p_grid = (50.0, 70.0, 85.0, 95.0)
    steps = min(args.steps, 5)
    LSR.search_layer(ctx, wt, ct, g, fmt, tabs, p_grid=p_grid, pack=True)          # warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        res = LSR.search_layer(ctx, wt, ct, g, fmt, tabs, p_grid=p_grid, pack=True)
    torch.cuda.synchronize()
    ms_step = (time.perf_counter() - t0) / steps * 1e3
    Nb = M * K // g
    evals = Nb * (6 + 6 * 5 + 2)                                       # block x atom evaluations of the scoring calls
    result = {
        "metric": "layer pair-search latency", "value": ms_step, "unit": "ms", "n_gpus": 1, "steps": steps, "warmup": 1,
        "ms_per_step": ms_step, "higher_is_better": False, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "full per-layer search of the C3 down-projection 4096x11008 bf16, g=16, UE4M3: 15 fixed pairs, "
                               "6 atoms x 4 values of p with a fitted second codebook, winner packed", "M": M, "K": K, "g": g,
                   "p_grid": list(p_grid)},
        "block_atom_evals_per_second": evals / (ms_step * 1e-3),
        "winner": {"kind": res.kind, "a": res.a, "b": res.b, "p_percent": res.p_percent, "acos": res.acos,
                   "best_fixed_pair_acos": float(res.acos_fixed.max())},
        "roofline": None,
    }
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    # the GPU raises its clock over the first 20-30 ms of load: the default warm-up covers that
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=300)
    ap.add_argument("--buffers", type=int, default=8)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--workload", default="pair_search", choices=["pair_search", "dd_histogram", "scale_histogram", "layer_scope", "finish", "model", "layer_search", "read_probe", "issue_probe"],
                    help="pair_search (default): the headline six-atom search; dd_histogram: the statistics pass of the "
                         "data-derived codebook on the same layer; scale_histogram: the statistics pass of the per-layer "
                         "scale shift on the same layer; layer_scope: E4M3 weights with one power-of-two scale for the layer; finish: block ranking and pools, "
                         "masked histogram and packing after a two-atom search; model: all 224 layers of a 7B-shaped "
                         "model in one call; layer_search: the whole per-layer procedure with the sweep over p")
    ap.add_argument("--config", default="C3_down", choices=["C1", "C2", "C3_up", "C3_down", "C5"],
                    help="layer of the pair_search workload (default: the headline down-projection)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run a plain copy kernel of known size (1 GiB read, 1 GiB written) a few times: the "
                         "reference the FETCH_SIZE / WRITE_SIZE counters are scaled by")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on one GPU only (no collectives, no sharding); use --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2605_14929_amd as sop
    import sop_inputs as si

    if args.workload == "read_probe":
        return bench_probe(args)
    if args.workload == "issue_probe":
        return bench_issue(args)
    if args.workload == "dd_histogram":
        return bench_dd(args)
    if args.workload == "scale_histogram":
        return bench_fl(args)
    if args.workload == "layer_scope":
        return bench_ls(args)
    if args.workload == "finish":
        return bench_finish(args)
    if args.workload == "model":
        return bench_model(args)
    if args.workload == "layer_search":
        return bench_layer_search(args)

    W, c, cfg = si.make_config(args.config)
    M, K, g = cfg["M"], cfg["K"], cfg["g"]
    A = len(cfg["atoms"])
    P = A * (A - 1) // 2
    Nb = M * K // g
    tabs = sop.build_alphabet(cfg["atoms"], bof_draws=si.normal_draws(1 << 20, 4242))
    fmt = sop.fmt_by_name(cfg["fmt"])
    headline = args.config == "C3_down"
    label = {"C1": "C1 layer 256x1024 fp32", "C2": "C2 attention projection 4096x4096 bf16 (outliers, row scales)",
             "C3_up": "C3 up-projection 11008x4096 bf16", "C3_down": "C3 down-projection 4096x11008 bf16",
             "C5": "C5 70B-shaped MLP layer 28672x8192 bf16"}[args.config]

    dev = torch.device("cuda", 0)
    w0 = torch.from_numpy(W).to(dev)
    if cfg["dtype"] == "bf16":
        w0 = w0.to(torch.bfloat16)
    esz = w0.element_size()
    if args.config == "C5":
        args.buffers = min(args.buffers, 2)
    bufs = [w0] + [torch.roll(w0, shifts=17 * i, dims=0).contiguous() for i in range(1, args.buffers)]
    ct = torch.from_numpy(c).to(dev)
    ctx = sop.Context(0)
    t0 = time.perf_counter()
    ctx.set_alphabet(tabs)
    alphabet_upload_ms = (time.perf_counter() - t0) * 1e3
    out = ctx.alloc_outputs(M, K, g, emit=False)

    if args.copy_calibration:
        src = torch.ones(1 << 28, dtype=torch.float32, device=dev)      # 1 GiB
        dst = torch.empty_like(src)
        for _ in range(4):
            torch.add(src, 1.0, out=dst)                                  # reads 2^30 B, writes 2^30 B
        torch.cuda.synchronize()
        del src, dst

    for i in range(args.warmup):
        ctx.pair_search(bufs[i % len(bufs)], ct, g, fmt, out=out)
    torch.cuda.synchronize()

    ms_step, ev_ms = timed_region(lambda i: ctx.pair_search(bufs[i % len(bufs)], ct, g, fmt, out=out), args.steps)
    last_pair = out.acos_pair.cpu().numpy()[:P].copy()
    # outside the timed region: the latency of single calls, each between its own pair of events
    n_lat = min(args.steps, 50)
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(n_lat)]
    for i in range(n_lat):
        ev[i][0].record()
        ctx.pair_search(bufs[i % len(bufs)], ct, g, fmt, out=out)
        ev[i][1].record()
    torch.cuda.synchronize()
    lat_ms = float(np.mean([a.elapsed_time(b) for a, b in ev]))
    lat_min_ms = float(np.min([a.elapsed_time(b) for a, b in ev]))
    lat_med_ms = float(np.median([a.elapsed_time(b) for a, b in ev]))

    # algorithmic HBM bytes of one launch: every weight once, the channel norms once, the
    # per-block selector words and the ACos vectors out
    sel_bytes = 2 if P <= 16 else 4                                       # one selector word per block
    alg_bytes = M * K * esz + K * 4 + Nb * sel_bytes + (A + P) * 8
    achieved = alg_bytes / (ev_ms * 1e-3) / 1e9
    n_groups = len({(float(t[0]), float(t[-1])) for t in tabs})           # atoms with equal endpoints share a scale
    n_copies = 0                                                          # atoms that are the sign-negated copy of an earlier atom
    for i, t in enumerate(tabs):
        if any(t.size == u.size and np.array_equal(t, -u[::-1]) for u in tabs[:i]):
            n_copies += 1
    if fmt.sign_bits:                                                     # a copy's group of mirrored endpoints is not prepared either
        n_groups = len({tuple(sorted((abs(float(t[0])), abs(float(t[-1]))))) for t in tabs})
    alg_ops = algorithmic_lane_ops(M * K, g, A, n_groups, P, signs=2 if fmt.sign_bits else 1, n_copies=n_copies)
    cff = counters_from_file() if headline else None

    # last step ran on buffer (steps-1) % n: check it against the oracle when that is buffer 0
    result = {
        "metric": "block x atom evaluations/sec", "value": Nb * A / (ms_step * 1e-3), "unit": "block*atom evals/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": f"{label}, g={g}, {cfg['fmt']}, {A} atoms ({','.join(cfg['atoms'])}), {P} pairs, search mode"
                               + (" (both signs of the scale tried per atom; an atom counts once)" if fmt.sign_bits else ""),
                   "M": M, "K": K, "g": g, "scale_format": cfg["fmt"], "atoms": list(cfg["atoms"]), "pairs": P,
                   "weight_dtype": cfg["dtype"], "buffers_rotated": len(bufs), "alphabet_upload_ms_once": alphabet_upload_ms},
        "layer_latency_ms": lat_ms, "layer_latency_median_ms": lat_med_ms, "layer_latency_min_ms": lat_min_ms,
        "counters_from_file": cff,
        # the six-atom search is bound by vector-ALU instruction issue (the method's lane-operations take 34 us per launch
        # at the full-rate peak and twice that at the rate three wavefronts per SIMD reach, against 12 us of algorithmic
        # HBM traffic); the HBM view of the same launch is given beside it
        "roofline": {"bound": "alu", "achieved": alg_ops / (ev_ms * 1e-3) / 1e12, "peak": VALU_PEAK_TLOPS, "unit": "T lane-ops/s",
                     "frac": alg_ops / (ev_ms * 1e-3) / 1e12 / VALU_PEAK_TLOPS, "traffic": parse_traffic() if headline else None,
                     "traffic_source": "profiles/search_kernel_c3down_hbm_traffic.txt (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE, not measured in this run)" if headline else None,
                     "frac_of_half_rate_class_peak": alg_ops / (ev_ms * 1e-3) / 1e12 / VALU_HALF_RATE_TLOPS,
                     "op_definition": "fp32 lane-operations of the method's arithmetic, an fma counted once; peak = the published 157.3 TFLOP/s / 2 "
                                      "= 256 CU x 4 SIMD x 32 lanes/clock x 2.4 GHz (a SIMD takes plain register-operand arithmetic from two wavefronts at a "
                                      "time; compares, min/max, conversions, 3-operand integer forms and scalar-operand forms go one at a time, 39.3)",
                     "algorithmic_lane_ops_per_launch": alg_ops, "algorithmic_lane_ops_per_weight": alg_ops / (M * K),
                     "kernel": "sopk::search_kernel", "event_ms_per_launch": ev_ms},
        "roofline_hbm": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                         "frac": achieved / HBM_PEAK_GBS, "target_frac": 0.60, "algorithmic_bytes_per_launch": alg_bytes},
    }

    if not args.no_cpu_baseline:
        from oracle import pairsearch as ops
        rows = M
        ofmt = ops.make_fmt(fmt.sign_bits, fmt.exp_bits, fmt.man_bits, fmt.container_bits, fmt.bias, fmt.max_code)
        t0 = time.perf_counter()
        ref = ops.pair_search(W[:rows], c, tabs, g, ofmt, want_codes=False)
        dt = time.perf_counter() - t0
        result["cpu_baseline"] = {"value": rows * (K // g) * A / dt, "unit": "block*atom evals/s", "cores": ops.num_threads(),
                                  "kind": "oracle", "sample": f"the whole layer ({rows} rows), OpenMP over rows, {dt:.2f} s wall"}
        t0 = time.perf_counter()
        ops.pair_search(W[:256], c, tabs, g, ofmt, want_codes=False, n_threads=1)
        dt1 = time.perf_counter() - t0
        result["cpu_baseline_one_thread"] = {"value": 256 * (K // g) * A / dt1, "unit": "block*atom evals/s", "cores": 1, "kind": "oracle",
                                             "sample": f"the first 256 rows, one thread, {dt1:.2f} s wall"}
        # parity of the benchmarked configuration in the same run (buffer 0)
        chk = ctx.pair_search(bufs[0], ct, g, fmt, out=out)
        torch.cuda.synchronize()
        d_acos = float(np.max(np.abs(chk.acos_pair.cpu().numpy()[:P] - ref.acos_pair)))
        sel_ok = bool(np.array_equal(chk.sel_words.cpu().numpy().view(np.uint16).astype(np.uint32), ref.sel_words))
        result["parity_in_run"] = {"max_abs_dACos": d_acos, "selector_bits_equal": sel_ok}
    result["untimed_clock_ramp_ms"] = CLOCK_RAMP_MS
    print(json.dumps(result))
    sys.stdout.flush()
    ctx.close()


if __name__ == "__main__":
    main()
