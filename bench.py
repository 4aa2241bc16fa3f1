#!/usr/bin/env python3
"""Benchmark of the STaMP quantized linear forward on one MI355X.

One "step" is one call of stamp_linear_forward (sequence Haar transform + mixed-precision
quantization + integer GEMM on the matrix cores + dequantization + inverse transform + bf16 store)
over one batch of seeded synthetic input that is already resident in HBM.  Prints ONE JSON line:
the throughput of the whole step, the roofline of the dominant kernel (the GEMM over the 4-bit rows,
under the engine that the step ran with), the same kernel's figures under the other engine, the
transform + quantization stage against HBM, per-stage times, and the oracle timed on the host.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg5] [--engine fp6|int8] [--no-cpu-baseline]
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM_GBS = 8000.0        # MI355X HBM3E
PEAK_INT8_TOPS = 5000.0      # MI355X dense int8 MFMA, TOP/s
PEAK_FP6_TFLOPS = 10100.0    # MI355X dense fp6 MFMA, TFLOP/s


def log(msg):
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def stage_time_ms(fn, iters, torch):
    """Average duration of one launch sequence `fn`, HIP events on the current stream."""
    fn()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(iters):
        fn()
    e1.record()
    e1.synchronize()
    return e0.elapsed_time(e1) / iters


def read_traffic(engine, workload_name):
    """HBM bytes per launch of the engine's GEMM kernel from the committed rocprofv3 --pmc summary, if any."""
    path = os.path.join(ROOT, "profiles", f"gemm_lo_{engine}_{workload_name}_pmc.txt")
    try:
        for line in open(path):
            if line.startswith("traffic_bytes_per_launch:"):
                return float(line.split(":", 1)[1])
    except OSError:
        pass
    return None


def cpu_baseline(w, inp, ncols, nseq):
    """The oracle, as it stands, on a bounded sample: `nseq` sequences of the workload through the whole
    layer, the GEMM / dequantization / inverse on the first `ncols` output columns, that part's time
    scaled by d_out / ncols."""
    import numpy as np
    from oracle import stamp_oracle as so
    try:
        from threadpoolctl import threadpool_info
        threads = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        threads = os.cpu_count() or 1
    nseq = min(nseq, w.batch)
    X = inp["X_f32"][:nseq]
    t0 = time.perf_counter()
    qa = so.quantize_activation(X, w.xform, w.levels, w.k_hi, w.bits_hi, w.bits_lo, w.grid_h, w.grid_w,
                                act_quant=w.act_quant)
    t1 = time.perf_counter()
    qw, sw = so.quantize_weight(inp["W"][:, :ncols], w.bits_w)   # plan-time work, not counted
    t2 = time.perf_counter()
    so.linear_from_codes(qa["codes"], qa["scales"], qw, sw, w.xform, w.levels, w.grid_h, w.grid_w, zeros=qa.get("zeros"))
    t3 = time.perf_counter()
    t_total = (t1 - t0) + (t3 - t2) * (w.d_out / ncols)
    return {
        "value": nseq * w.seq_len / t_total, "unit": "tokens/s", "cores": int(threads), "kind": "oracle",
        "sample": (f"{nseq} of {w.batch} sequences ({nseq * w.seq_len} tokens): transform+quantization in full "
                   f"({t1 - t0:.2f} s, single-threaded numpy), integer GEMM (fp64 BLAS, {threads} threads) + "
                   f"dequantization + inverse on the first {ncols} of {w.d_out} output columns "
                   f"({t3 - t2:.2f} s, scaled x{w.d_out / ncols:.1f})"),
    }


def time_layer(st, torch, w, inp, args):
    """ms per stamp_linear_forward call of workload w (bf16 output), inputs generated by the caller."""
    Xd = st.to_device_x(inp, w)
    Wd = torch.from_numpy(inp["W"]).cuda()
    bd = None if inp.get("bias") is None else torch.from_numpy(inp["bias"]).cuda()
    plan = st.StampPlan(st.plan_desc_for(w, "bf16"), Wd, bd)
    ws = plan.alloc_workspace()
    Y = torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.int16, device="cuda")
    for _ in range(args.warmup):
        plan.linear_forward(Xd, Y, ws)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        plan.linear_forward(Xd, Y, ws)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / args.steps
    extra = {}
    if w.group_size:
        q_hi, q_lo, scales = plan.alloc_act_buffers()
        plan.quantize_act(Xd, q_hi, q_lo, scales, ws)
        extra["quantize_act_ms"] = stage_time_ms(lambda: plan.quantize_act(Xd, q_hi, q_lo, scales, ws), args.stage_iters, torch)
        fms = stage_time_ms(lambda: plan.linear_forward_q(q_hi, q_lo, scales, Y, ws), args.stage_iters, torch)
        extra["gemm_dequant_inverse_ms"] = fms
        extra["gemm_TOPs_lower_bound"] = 2.0 * w.batch * w.seq_len * w.d_in * w.d_out / (fms * 1e-3) / 1e12
    plan.destroy()
    del ws, Y, Xd, Wd
    return ms, extra


def general_path_variants(st, torch, args):
    """The settings served by the library's general path (transform level by level over fp32 buffers, inverse after the
    GEMM instead of in its epilogue), each next to the nearest fast-path plan on the same inputs:
    the language-model set-up of the paper's appendix (2048 tokens, 3 levels, 64 8-bit tokens, first token left out
    of the transform), the sequency-ordered WHT and the DCT on the same layer, the transformed-bias form, and per-block
    (64-channel) scales on the image-token layer (the set-up of the paper's LVM experiments)."""
    from dataclasses import replace
    import numpy as np
    from gen import get_workload, make_inputs
    out = {}

    def run(tag, base_w, base_inp, **kw):
        w = replace(base_w, **kw)
        ms, extra = time_layer(st, torch, w, base_inp, args)
        out[tag] = {"ms_per_step": ms, "tokens_per_s": w.batch * w.seq_len / (ms * 1e-3), **extra}
        log(f"variant {tag}: {ms:.3f} ms/step")

    w2 = get_workload("cfg2", levels=3)
    inp2 = make_inputs(w2, with_bias=True)
    run("llm_J3_fast_path", w2, inp2)
    run("llm_J3_first_token_left_out", w2, inp2, skip_first=True)
    run("llm_J3_transformed_bias", w2, inp2, bias_mode="transformed")
    run("llm_wht", w2, inp2, xform="wht", levels=0)
    run("llm_dct", w2, inp2, xform="dct", levels=0)
    out["llm_workload"] = f"B={w2.batch} s={w2.seq_len} d_in={w2.d_in} d_out={w2.d_out} k_hi={w2.k_hi}, bias, bf16 in/out"
    del inp2
    w4 = get_workload("cfg4", levels=3)
    inp4 = make_inputs(w4)
    run("lvm_J3_fast_path", w4, inp4)
    run("lvm_J3_per_block_scales", w4, inp4, group_size=64)
    out["lvm_workload"] = f"B={w4.batch} s={w4.seq_len} (64x64 grid) d_in={w4.d_in} d_out={w4.d_out} k_hi={w4.k_hi}, bf16 in/out"
    del inp4
    # the language-model setting on longer sequences: 3 levels leave 512 approximations per sequence (fast path, no top levels)
    w3 = get_workload("cfg3", levels=3)
    inp3 = make_inputs(w3)
    run("llm_J3_4096_tokens_fast_path", w3, inp3)
    out["llm_4096_workload"] = f"B={w3.batch} s={w3.seq_len} d_in={w3.d_in} d_out={w3.d_out} k_hi={w3.k_hi}, bf16 in/out"
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="cfg5")
    ap.add_argument("--stage-iters", type=int, default=10)
    ap.add_argument("--cpu-cols", type=int, default=16384)
    ap.add_argument("--cpu-seqs", type=int, default=4)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-variants", action="store_true",
                    help="skip the measurements of the general-path settings (first token left out, WHT, DCT, "
                         "transformed bias, per-block scales)")
    ap.add_argument("--unfused", action="store_true")
    ap.add_argument("--engine", choices=["int8", "fp6"], default="fp6",
                    help="matrix pipeline of the 4-bit rows' GEMM (the library's default is fp6)")
    ap.add_argument("--act-quant", choices=["sym", "asym"], default="sym",
                    help="activation quantizer: symmetric absmax (the benchmark configurations) or the paper's "
                         "asymmetric min-max form")
    ap.add_argument("--d-in", type=int, default=0, help="override the workload's d_in (e.g. the layer that follows it)")
    ap.add_argument("--d-out", type=int, default=0, help="override the workload's d_out")
    ap.add_argument("--levels", type=int, default=0, help="override the transform depth (the paper's experiments use 3)")
    ap.add_argument("--skip-first", action="store_true", help="leave the first token out of the transform (general path)")
    ap.add_argument("--xform", choices=["haar1d", "haar2d", "wht", "dct", "identity"], default=None,
                    help="override the sequence transform (wht, dct: general path)")
    ap.add_argument("--bias-mode", choices=["after", "transformed"], default="after")
    ap.add_argument("--group-size", type=int, default=0, help="64: per-block scales (general path)")
    ap.add_argument("--calib-copy", action="store_true",
                    help="also run one plain elementwise kernel that reads 1 GiB and writes 1 GiB (int32 add), the "
                         "known-size reference for scaling rocprofv3 FETCH_SIZE / WRITE_SIZE readings")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: this build runs the STaMP linear layer on ONE GPU; --gpus N with N > 1 is not "
              "supported (sequences are independent: the batch would be sharded without communication).",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    import paper_2510_26771_amd as st
    from gen import get_workload, make_inputs

    st.load_library()
    assert torch.cuda.is_available(), "bench.py needs a GPU"
    over = {k: v for k, v in (("d_in", args.d_in), ("d_out", args.d_out), ("levels", args.levels)) if v > 0}
    if args.skip_first:
        over["skip_first"] = True
    if args.xform:
        over["xform"] = args.xform
        if args.xform in ("wht", "dct", "identity"):
            over["levels"] = 0
    if args.bias_mode != "after":
        over["bias_mode"] = args.bias_mode
    if args.group_size:
        over["group_size"] = args.group_size
    w = get_workload(args.workload, act_quant=args.act_quant, **over)
    general = bool(w.skip_first or w.xform in ("wht", "dct") or w.bias_mode != "after" or w.group_size
                   or (w.xform == "haar1d" and w.seq_len & (w.seq_len - 1)))
    log(f"generating {w.name}: B={w.batch} s={w.seq_len} d_in={w.d_in} d_out={w.d_out}")
    inp = make_inputs(w, with_bias=w.bias_mode != "after")
    Xd = st.to_device_x(inp, w)
    Wd = torch.from_numpy(inp["W"]).cuda()
    plan = st.StampPlan(st.plan_desc_for(w, "bf16"), Wd, None if inp["bias"] is None else torch.from_numpy(inp["bias"]).cuda())
    torch.cuda.synchronize()
    del Wd
    if args.unfused:
        plan.set_unfused(True)
    plan.set_gemm_engine(args.engine)
    ws = plan.alloc_workspace()
    Y = torch.empty((w.batch, w.seq_len, w.d_out), dtype=torch.int16, device="cuda")

    def step():
        plan.linear_forward(Xd, Y, ws)

    if not general:
        # a Haar setting without the fast path's block structure (e.g. more than 256 approximations) is served by the
        # general path as well: the library then refuses to launch single stages
        probe = plan.alloc_act_buffers()
        try:
            plan.debug_run_stage(0, Xd, *probe, Y, ws)
        except st.StampError as e:
            if e.status != 3:  # STAMP_ERR_UNSUPPORTED
                raise
            general = True
        torch.cuda.synchronize()
        del probe

    if args.calib_copy:
        src = torch.ones(1 << 28, dtype=torch.int32, device="cuda")
        dst = torch.empty_like(src)
        torch.add(src, 1, out=dst)
        torch.cuda.synchronize()
        del src, dst
    log("warmup")
    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # exactly K steps between two synchronizations (ms_per_step, value); an event between consecutive steps on
    # the launch stream gives every step's own duration as well (median / min / max)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    t0 = time.perf_counter()
    evs[0].record()
    for i in range(args.steps):
        step()
        evs[i + 1].record()
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    ms_per_step = (t1 - t0) * 1e3 / args.steps
    per_step = sorted(evs[i].elapsed_time(evs[i + 1]) for i in range(args.steps))
    step_stats = {"median": per_step[len(per_step) // 2], "min": per_step[0], "max": per_step[-1]}
    tokens = w.batch * w.seq_len
    log(f"{ms_per_step:.3f} ms/step (events: median {step_stats['median']:.3f}, min {step_stats['min']:.3f}, "
        f"max {step_stats['max']:.3f})")

    if general:
        # settings of the general path: no separately launchable stages; per-kernel times come from a kernel trace
        print(json.dumps({
            "metric": "tokens/sec through STaMP linear fwd", "value": tokens / (ms_per_step * 1e-3), "unit": "tokens/s",
            "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
            "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "int8" if w.group_size else args.engine,
            "data": "synthetic", "ms_per_step_events": step_stats,
            "config": {"workload": f"{w.name}: B={w.batch} s={w.seq_len} d_in={w.d_in} d_out={w.d_out} {w.xform} "
                                   f"J={w.levels} k_hi={w.k_hi} skip_first={w.skip_first} bias_mode={w.bias_mode} "
                                   f"group_size={w.group_size}", "path": "general"},
            "roofline": None, "cpu_baseline": None}), flush=True)
        plan.destroy()
        return

    # ---- per-stage timings (HIP events on the launch stream) ----
    q_hi, q_lo, scales = plan.alloc_act_buffers()
    plan.quantize_act(Xd, q_hi, q_lo, scales, ws)

    def run_stage(sid):
        return stage_time_ms(lambda: plan.debug_run_stage(sid, Xd, q_hi, q_lo, scales, Y, ws), args.stage_iters, torch)

    stages = {}
    names = {0: "transform_quant_lo", 1: "transform_quant_hi", 2: "gemm_hi", 3: "inverse_top"}
    if args.engine == "fp6":
        names[6] = "repack_fp6"
    names[4] = "gemm_lo"
    if args.unfused:
        names[5] = "inverse_bottom"
    for sid, nm in names.items():
        stages[nm] = run_stage(sid)
    stages["quantize_act"] = stage_time_ms(lambda: plan.quantize_act(Xd, q_hi, q_lo, scales, ws), args.stage_iters, torch)
    log("stages ms: " + ", ".join(f"{k}={v:.4f}" for k, v in stages.items()))

    # the GEMM over the 4-bit rows under either engine.  Algorithmic work: 2 * rows * d_in * d_out operations
    lo_rows = w.batch * (w.seq_len - w.k_hi)
    gemm_ops = 2.0 * lo_rows * w.d_in * w.d_out
    epi = ", dequant only)" if args.unfused else ", fused dequant + in-block inverse)"

    def gemm_roofline(engine, ms):
        peak = PEAK_FP6_TFLOPS if engine == "fp6" else PEAK_INT8_TOPS
        achieved = gemm_ops / (ms * 1e-3) / 1e12
        sustained = st.mfma_rate(engine)
        return {"bound": "mfma", "achieved": achieved, "peak": peak, "unit": "TFLOP/s" if engine == "fp6" else "TOP/s",
                "frac": achieved / peak, "traffic": read_traffic(engine, w.name),
                "kernel": ("k_gemm6 (fp6 MFMA" if engine == "fp6" else "k_gemm (int8 MFMA") + ", 4-bit rows" + epi,
                "ops_per_launch": gemm_ops, "avg_launch_ms": ms,
                "mfma_only_rate_measured": sustained, "frac_of_mfma_only_rate": achieved / sustained if sustained else None}

    roofline = gemm_roofline(args.engine, stages["gemm_lo"])
    other = "int8" if args.engine == "fp6" else "fp6"
    plan.set_gemm_engine(other)
    if other == "fp6":
        run_stage(6)
    other_ms = run_stage(4)
    plan.set_gemm_engine(args.engine)
    roofline_other = gemm_roofline(other, other_ms)
    log(f"gemm_lo under the {other} engine: {other_ms:.4f} ms")
    # transform + quantization stage against the HBM roofline: X read + packed codes + scales written
    xbytes = 2 if w.x_dtype == "bf16" else 4
    qa_bytes = (w.batch * w.seq_len * w.d_in * xbytes + w.batch * w.k_hi * w.d_in
                + w.batch * (w.seq_len - w.k_hi) * w.d_in // 2 + w.batch * w.seq_len * 4)
    qa_gbs = qa_bytes / (stages["quantize_act"] * 1e-3) / 1e9
    lo_bytes = (w.batch * w.seq_len * w.d_in * xbytes + w.batch * (w.seq_len - w.k_hi) * w.d_in // 2
                + w.batch * (w.seq_len - w.k_hi) * 4 + w.batch * w.k_hi * w.d_in * 4)
    lo_gbs = lo_bytes / (stages["transform_quant_lo"] * 1e-3) / 1e9
    roofline_quant = {"bound": "hbm", "achieved": qa_gbs, "peak": PEAK_HBM_GBS, "unit": "GB/s",
                      "frac": qa_gbs / PEAK_HBM_GBS, "bytes_per_call": qa_bytes,
                      "stage": "stamp_quantize_act (3 kernels)",
                      "dominant_kernel": {"name": "k_bottom", "achieved": lo_gbs, "frac": lo_gbs / PEAK_HBM_GBS,
                                          "bytes_per_launch": lo_bytes, "avg_launch_ms": stages["transform_quant_lo"]}}

    # The same layer without the sequence transform (identity plan: per-token quantization of X itself, the same
    # k tokens at 8 bits, same GEMM engines and epilogue stores): what the transform and its inverse cost here.
    # The paper reports this cost only as +4.8 % latency of one whole denoising step on an A100 (3-level DWT around
    # floating-point layers), so its figure is context, not a baseline for this number.
    from dataclasses import replace as _replace
    wi = _replace(w, xform="identity", levels=0, grid_h=0, grid_w=0)
    plan_i = st.StampPlan(st.plan_desc_for(wi, "bf16"), torch.from_numpy(inp["W"]).cuda())
    plan_i.set_gemm_engine(args.engine)
    ws_i = plan_i.alloc_workspace()
    for _ in range(args.warmup):
        plan_i.linear_forward(Xd, Y, ws_i)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        plan_i.linear_forward(Xd, Y, ws_i)
    torch.cuda.synchronize()
    ident_ms = (time.perf_counter() - t0) * 1e3 / args.steps
    plan_i.destroy()
    del ws_i
    log(f"same layer without the sequence transform: {ident_ms:.3f} ms/step")
    transform_cost = {"ms_per_step_without_transform": ident_ms, "overhead_frac": ms_per_step / ident_ms - 1.0,
                      "what": "identity plan: same quantizer, bit allocation, GEMM engine and stores, no Haar transform / inverse"}

    per_block = None
    if not args.no_variants:
        per_block = general_path_variants(st, torch, args)

    out = {
        "metric": "tokens/sec through STaMP linear fwd", "value": tokens / (ms_per_step * 1e-3), "unit": "tokens/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "fp6" if args.engine == "fp6" else "int8", "data": "synthetic",
        "config": {"workload": f"{w.name}: B={w.batch} s={w.seq_len} d_in={w.d_in} d_out={w.d_out} "
                               f"{w.xform} J={w.levels} k_hi={w.k_hi} W4A4(+{w.k_hi} int8 tokens), bf16 in/out",
                   "path": "unfused" if args.unfused else "fused", "gemm_engine": args.engine,
                   "act_quant": args.act_quant},
        "roofline": roofline, f"roofline_{other}_engine": roofline_other, "roofline_quant": roofline_quant,
        "ms_per_step_events": step_stats,
        "stages_ms": stages,
        "stages_note": ("each stage launched alone, back to back with itself, timed with HIP events; inside a step the "
                        "kernels follow each other on one stream and a kernel's first workgroups start while the "
                        "last ones of the kernel before it drain, so the stages add up to more than ms_per_step"),
        "transform_cost": transform_cost,
    }
    if per_block is not None:
        out["general_path_variants"] = per_block
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle)")
        out["cpu_baseline"] = cpu_baseline(w, inp, min(args.cpu_cols, w.d_out), args.cpu_seqs)
    plan.destroy()
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
