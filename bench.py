#!/usr/bin/env python3
"""Benchmark of the Shampoo preconditioner hot path on one MI355X.

Workload (the configuration the headline metric is quoted on): every 2-D gradient of a 1.1B
LLaMA-style model (d=2048, 22 layers, FFN 5632, vocab 32000; 1 099 956 224 parameters) blocked
at <= 1024 x 1024 -> 1184 blocks, 2368 Kronecker factors; synthetic bf16 gradients with
power-law singular values (sigma_i ~ 1/i), beta = 0.95, eps = 1e-6 lambda_max.

One "step" = one pass of the whole path over that batch, inputs resident in HBM:
    asteria_stats_update (all blocks) -> asteria_inverse_root (all factors, the "full
    preconditioner refresh") -> asteria_precondition (all blocks).
`value` = milliseconds per full refresh (the inverse-root call over all factors);
`ms_per_step` = the whole pass.  Prints ONE JSON line on stdout; progress goes to stderr.

Further objects of the same line: `soap` (the SOAP variant on the same model, blocks <= 2048),
`lowrank_batch` (64 blocks of 1024 x 1024, rank-32 + noise), `stress_4096` (8 blocks of 4096 x 4096,
singular values over 8 decades, eps = 1e-8 lambda_max), `staleness` (the refresh on a second
stream behind the steps, bounded staleness S) and `cpu_baseline` (the float64 oracle timed on the
host cores).  `--sections` selects them.
"""
from __future__ import annotations

import argparse
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_F32_MFMA = 157.3   # TFLOP/s, MI355X dense fp32 matrix
PEAK_F64_MFMA = 78.6    # TFLOP/s, MI355X dense fp64 matrix
PEAK_BF16_MFMA = 2500.0 # TFLOP/s, MI355X dense bf16 and fp16 matrix
PEAK_I8_MFMA = 5000.0   # TOP/s, MI355X dense int8 matrix
# What a register-only loop of v_mfma_f64_16x16x4_f64 with random operands sustains on the box
# (2 or 4 wavefronts per SIMD, 8 independent accumulators each, 2.38 GHz): context for the fp64
# kernel's fraction of the published peak, never used as `peak`.
MEASURED_F64_MFMA_LOOP = 58.8
PEAK_HBM = 8000.0       # GB/s

ALL_SECTIONS = ("shampoo", "cpu", "soap", "lowrank", "stress", "staleness")


def stored_traffic(key: str):
    """HBM bytes per WORKING launch measured with rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE on this
    workload (each scaled by a plain copy of known size); the runs and their summary live under
    profiles/ (a launch that finds every factor finished moves no data and is left out)."""
    path = os.path.join(ROOT, "profiles", "gemm_grouped__llama1b_b1024_hbm_traffic.md")
    try:
        m = re.search(rf"{key}\s*=\s*([0-9.eE+-]+)", open(path).read())
        return float(m.group(1)) if m else None
    except OSError:
        return None


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def sym_gemm_flops(n: int) -> float:
    """Algorithmic flops of one symmetric n x n x n product when only one triangle is computed."""
    return float(n) * (n + 1) * n


class RootRun:
    """One inverse-root workload: statistics, roots and preconditioned gradients of a list of blocks,
    timed stage by stage with events on the stream the library launches on, every grouped-GEMM
    launch bracketed by the library's own events."""

    def __init__(self, torch, ast, Gs, shapes, beta, eps_rel, opts, ws_gib, acc=0):
        self.torch, self.ast = torch, ast
        dev = Gs[0].device
        self.shapes, self.beta, self.eps_rel, self.opts = shapes, beta, eps_rel, opts
        self.Gs = Gs
        self.Ls = [torch.zeros(m, m, device=dev) for m, n in shapes]
        self.Rs = [torch.zeros(n, n, device=dev) for m, n in shapes]
        self.XLs = [torch.empty(m, m, device=dev) for m, n in shapes]
        self.XRs = [torch.empty(n, n, device=dev) for m, n in shapes]
        self.Ps = [torch.empty(m, n, device=dev) for m, n in shapes]
        self.blocks = ast.Blocks([(G, L, R, acc) for G, L, R in zip(Gs, self.Ls, self.Rs)])
        self.factors = ast.Factors([(L, X) for L, X in zip(self.Ls, self.XLs)] + [(R, X) for R, X in zip(self.Rs, self.XRs)])
        self.pblocks = ast.PBlocks(list(zip(self.XLs, Gs, self.XRs, self.Ps)))
        self.nf = len(self.factors)
        self.fsize = [m for m, n in shapes] + [n for m, n in shapes]
        self.full, mn = ast.inverse_root_workspace_bytes(self.factors, opts)
        self.ws_bytes = int(max(min(self.full, ws_gib * 2**30), mn, ast.precondition_workspace_bytes(self.pblocks),
                                ast.stats_update_workspace_bytes(self.blocks)))
        self.ws = torch.empty(self.ws_bytes, dtype=torch.uint8, device=dev)
        self.info = torch.zeros(self.nf, dtype=torch.int32, device=dev)
        self.iters = torch.zeros(self.nf, dtype=torch.int32, device=dev)
        self.resid = torch.zeros(self.nf, device=dev)
        self.plan = ast.inverse_root_plan(eps_rel, relative=True, root=4, opts=opts)

    def step(self, ev=None):
        ast = self.ast
        if ev: ev[0].record()
        ast.stats_update(self.blocks, self.beta, ws=self.ws)
        if ev: ev[1].record()
        ast.inverse_root(self.factors, self.eps_rel, relative=True, root=4, opts=self.opts, info=self.info,
                         iters=self.iters, resid=self.resid, ws=self.ws)
        if ev: ev[2].record()
        ast.precondition(self.pblocks, ws=self.ws)
        if ev: ev[3].record()

    def timed(self, steps, warmup, tag):
        torch, ast = self.torch, self.ast
        for w in range(warmup):
            t = time.time()
            self.step()
            torch.cuda.synchronize()
            log(f"[bench] {tag} warmup {w}: {1e3 * (time.time() - t):.0f} ms")
        evs = [[torch.cuda.Event(enable_timing=True) for _ in range(4)] for _ in range(steps)]
        ast.profile_enable(200000)
        torch.cuda.synchronize()
        t_wall = time.time()
        for s in range(steps):
            self.step(evs[s])
            torch.cuda.synchronize()          # step boundary (also lets the iteration counts be read)
            log(f"[bench] {tag} step {s}: {evs[s][0].elapsed_time(evs[s][3]):.0f} ms")
        wall_ms = 1e3 * (time.time() - t_wall)
        i8f = ast.profile_i8_flops()         # products of the prefix by where the device sent them
        pair_flops, i8_ops = ast.profile_root_work()
        prof = ast.profile_collect(200000)
        ms = lambda a, b: sum(e[a].elapsed_time(e[b]) for e in evs) / steps
        return dict(stats_ms=ms(0, 1), refresh_ms=ms(1, 2), precond_ms=ms(2, 3), step_ms=ms(0, 3), wall_ms=wall_ms,
                    prof=prof, pair_flops=pair_flops, i8_ops=i8_ops, i8_flops=i8f, info=self.info.cpu().numpy(), iters=self.iters.cpu().numpy())


def gemm_rooflines(res, steps, step_ms, headline=False):
    """Per GEMM kernel of the refresh: algorithmic flops its launches executed / the sum of their
    durations, against the published dense peak of the instruction it issues.  A launch that found
    every factor finished (or, for the fp64 fall-back grid, every product taken by the int8 path)
    does no work; such launches are counted and their (microsecond) durations left out of the rates.
    `avg_launch_ms` is the mean over the launches that worked, `avg_launch_ms_all` the mean over every launch
    (what a profiler's per-kernel average shows)."""
    # the stored HBM bytes are those of the headline workload
    traffic_of = stored_traffic if headline else (lambda key: None)
    prof, pair_flops, i8_ops, i8f = res["prof"], res["pair_flops"], res["i8_ops"], res["i8_flops"]
    def split(kinds):
        ms = [t for t, k in prof if k in kinds]
        top = max(ms, default=0.0)
        work = [t for t in ms if t > 0.05 * top]          # an empty grid takes ~0.1 ms, a working launch 5 - 50
        return ms, work
    out, shares = {}, {}
    # every product is counted on the device where it ran (runs with pinned precision options are not)
    f64_cores, f_i8_4, f_i8_5 = i8f
    all64, w64 = split((1,))
    all16, w16 = split((224,))
    all8, w8 = split((304, 305))
    t64, t16, t8 = (sum(x) * 1e-3 for x in (w64, w16, w8))
    if w64 and f64_cores > 0:
        tf = f64_cores / t64 / 1e12
        out["roofline_fp64"] = {"kernel": "gemm_grouped_kernel<double> (products of the leading root iterations on the fp64 matrix cores)",
                                "bound": "mfma", "achieved": round(tf, 2), "peak": PEAK_F64_MFMA, "unit": "TFLOP/s",
                                "frac": round(tf / PEAK_F64_MFMA, 4), "traffic": traffic_of("traffic_bytes_per_launch_fp64"),
                                "instruction_loop_tflops_measured": MEASURED_F64_MFMA_LOOP,
                                "launches": len(all64), "working_launches": len(w64),
                                "avg_launch_ms": round(1e3 * t64 / len(w64), 4), "avg_launch_ms_all": round(sum(all64) / len(all64), 4), "flops_per_launch": round(f64_cores / len(w64), 1)}
        shares["roofline_fp64"] = t64
    if w16 and pair_flops > 0:
        tf = pair_flops / t16 / 1e12
        out["roofline_split_fp16"] = {
            "kernel": "pair_product_kernel (X updates and the root iterations after the prefix: operands stored as two fp16 "
                      "terms, 3 fp16 MFMA passes per product)",
            "bound": "mfma", "achieved": round(3 * tf, 2), "peak": PEAK_BF16_MFMA, "unit": "TFLOP/s (fp16 MFMA issued)",
            "frac": round(3 * tf / PEAK_BF16_MFMA, 4),
            "fp32_equivalent_tflops": round(tf, 2), "useful_frac": round(tf / PEAK_BF16_MFMA, 4),
            "traffic": traffic_of("traffic_bytes_per_launch_fp16"), "launches": len(all16), "working_launches": len(w16),
            "avg_launch_ms": round(1e3 * t16 / len(w16), 4), "avg_launch_ms_all": round(sum(all16) / len(all16), 4), "flops_per_launch": round(3 * pair_flops / len(w16), 1)}
        shares["roofline_split_fp16"] = t16
    if w8 and f_i8_4 + f_i8_5 > 0:
        ops = i8_ops                                       # 10 or 13 int8 MFMA passes per product with 4 digits, 15 or 19 with 5
        useful = f_i8_4 + f_i8_5
        out["roofline_int8_slices"] = {
            "kernel": "digit_product_kernel<4 | 5> (products of the leading iterations: operands as 32- or 40-bit integers in "
                      "base-256 digits, 10 to 19 int8 MFMA passes per product, exact int32 sums, fp64 assembly; digits and levels "
                      "are chosen per factor on the device and the work counted there)",
            "bound": "mfma", "achieved": round(ops / t8 / 1e12, 2), "peak": PEAK_I8_MFMA, "unit": "TOP/s (int8 MFMA issued)",
            "frac": round(ops / t8 / 1e12 / PEAK_I8_MFMA, 4),
            "fp64_equivalent_tflops": round(useful / t8 / 1e12, 2), "useful_frac": round(useful / t8 / 1e12 / PEAK_I8_MFMA, 4),
            "flops_share_4_digits": round(f_i8_4 / useful, 4), "flops_share_5_digits": round(f_i8_5 / useful, 4),
            "flops_share_declined_to_fp64_cores": round(f64_cores / (useful + f64_cores), 6),
            "traffic": traffic_of("traffic_bytes_per_launch_int8"), "launches": len(all8), "working_launches": len(w8),
            "avg_launch_ms": round(1e3 * t8 / len(w8), 4), "avg_launch_ms_all": round(sum(all8) / len(all8), 4), "flops_per_launch": round(ops / len(w8), 1)}
        shares["roofline_int8_slices"] = t8
    out["gemm_time_share_ms_per_step"] = {k.replace("roofline_", ""): round(1e3 * v / steps, 1) for k, v in shares.items()}
    if not shares:                                        # pinned precision options
        out["refresh_mfma"] = None
        return out
    dominant = max(shares, key=shares.get)
    out["roofline"] = dict(out[dominant], time_share_of_step=round(1e3 * shares[dominant] / steps / step_ms, 4))
    # the refresh as a whole: every kernel's fraction of its own peak weighted by its time, the time
    # outside GEMM kernels (slicing, lambda_max estimate, start, hand-over, control) counting as zero
    refresh_ms = res["refresh_ms"]
    in_gemm = sum(1e3 * v / steps for v in shares.values())
    weighted = sum(out[k]["frac"] * 1e3 * shares[k] / steps for k in shares) / refresh_ms
    useful = sum(out[k].get("useful_frac", out[k]["frac"]) * 1e3 * shares[k] / steps for k in shares) / refresh_ms
    out["refresh_mfma"] = {"issued_frac_time_weighted": round(weighted, 4), "useful_frac_time_weighted": round(useful, 4),
                           "ms_in_gemm_kernels": round(in_gemm, 1), "ms_outside_gemm_kernels": round(refresh_ms - in_gemm, 1)}
    return out


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=3)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--ws-gib", type=float, default=128.0, help="workspace handed to the library (a single pass needs about 66 GiB)")
    ap.add_argument("--max-blocks", type=int, default=0, help="debug: truncate the batch")
    ap.add_argument("--fp64-iters", type=int, default=-1)
    ap.add_argument("--lowp-from", type=int, default=-1, help="first iteration on the fp16 cores with split operands (-1 = library rule)")
    ap.add_argument("--int8-slices", type=int, default=-1, help="products of the fp64 iterations: -1 = library default (int8 cores, 5 slices), 0 = fp64 cores, 4 | 5")
    ap.add_argument("--schedule", type=int, default=1, help="1 = interval-adapted coefficients, 0 = classical Newton")
    ap.add_argument("--sections", default=",".join(ALL_SECTIONS),
                    help="comma-separated subset of " + ",".join(ALL_SECTIONS) + " (shampoo always runs)")
    ap.add_argument("--soap-groups", type=int, default=2, help="auxiliary streams the SOAP refresh deals its factors to (1..4)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-soap", action="store_true", help="skip the SOAP section (blocks <= 2048)")
    ap.add_argument("--save-inputs", default="", help="generate the headline workload's gradients, write them to this file and exit")
    ap.add_argument("--load-inputs", default="", help="read the gradients from a file written by --save-inputs instead of generating "
                    "them (runs under hardware counters: the process then launches no generator kernels)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one plain 1 GiB device copy (reference for rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU; --gpus N with N > 1 is not supported "
              "(no collectives or sharding in this library).", file=sys.stderr)
        return 2
    sections = set(s for s in args.sections.split(",") if s)
    if args.no_cpu_baseline: sections.discard("cpu")
    if args.no_soap: sections.discard("soap")

    import torch
    import paper_2605_16184_amd as ast
    from paper_2605_16184_amd import workloads as W

    dev = "cuda:0"
    torch.cuda.set_device(0)
    beta, eps_rel = 0.95, 1e-6

    shapes = W.block_shapes(W.llama_1b_matrices(), 1024)
    if args.max_blocks:
        shapes = shapes[:: max(1, len(shapes) // args.max_blocks)][: args.max_blocks]
    by_shape, by_factor, params = W.census(shapes)
    log(f"[bench] {len(shapes)} blocks, factors {by_factor}, {params} parameters")

    t0 = time.time()
    # the orthogonal templates are factorised by the host's LAPACK: the same inputs then serve runs
    # under hardware counters, which keep the device's solver library out of the process
    if args.load_inputs:
        flat = torch.load(args.load_inputs, weights_only=True)["G"].to(dev)
        Gs, off = [], 0
        for m, n in shapes:
            Gs.append(flat[off:off + m * n].view(m, n))
            off += m * n
        assert off == flat.numel(), "the file holds another batch"
    else:
        Gs = W.powerlaw_blocks(shapes, dev, bank=W.TemplateBank(dev, qr_on_host=True))
    if args.save_inputs:
        torch.save({"G": torch.cat([g.reshape(-1) for g in Gs]).cpu()}, args.save_inputs)
        log(f"[bench] gradients written to {args.save_inputs}")
        return 0
    opts = ast.RootOpts(fp64_iters=args.fp64_iters, schedule=args.schedule, lowp_from=args.lowp_from,
                        int8_slices=args.int8_slices)
    run = RootRun(torch, ast, Gs, shapes, beta, eps_rel, opts, args.ws_gib)
    torch.cuda.synchronize()
    log(f"[bench] inputs generated in {time.time() - t0:.1f} s; {torch.cuda.memory_allocated() / 2**30:.1f} GiB resident; "
        f"workspace {run.ws_bytes / 2**30:.1f} GiB (single pass would need {run.full / 2**30:.1f} GiB)")

    if args.calibrate_copy:
        src = torch.empty(2**28, dtype=torch.float32, device=dev).fill_(1.0)    # 1 GiB
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst

    res = run.timed(args.steps, args.warmup, "1.1B")
    j64, jlow, xt_lowp = run.plan
    stats_ms, refresh_ms, precond_ms, step_ms = res["stats_ms"], res["refresh_ms"], res["precond_ms"], res["step_ms"]
    it, info_h = res["iters"], res["info"]
    nf = run.nf
    stats_flops = sum(sym_gemm_flops(m) / m * n + sym_gemm_flops(n) / n * m for m, n in shapes)
    stats_bytes = sum(2 * m * n + 8 * (m * m + n * n) for m, n in shapes)
    precond_flops = sum(2.0 * m * n * (m + n) for m, n in shapes)
    precond_issued = sum(2.0 * (2.0 * m * n * n) + 3.0 * (2.0 * m * m * n) for m, n in shapes)
    precond_bytes = sum(4 * m * m + 4 * n * n + 2 * m * n + 4 * m * n for m, n in shapes)
    log(f"[bench] stats {stats_ms:.2f} ms  refresh {refresh_ms:.1f} ms  precondition {precond_ms:.2f} ms")
    log(f"[bench] Newton iterations min/mean/max {it.min()}/{it.mean():.1f}/{it.max()}, info!=0: {(info_h != 0).sum()}")

    out = {
        "metric": "ms per full preconditioner refresh (1B model) + % MFMA peak; ms per step",
        "value": round(refresh_ms, 3),
        "unit": f"ms per full refresh (inverse 4th roots of all {nf} factors)",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(step_ms, 3),
        "higher_is_better": False,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": "1.1B LLaMA-style model, all 2-D grads blocked at <=1024 (1184 blocks, 2368 factors), "
                               "bf16 power-law gradients, fp32 statistics, eps=1e-6*lambda_max, beta=0.95",
                   "blocks": len(shapes), "factors": nf,
                   "arithmetic": "fp32 storage; statistics: bf16 MFMA, fp32 sums; roots: the leading iterations as 32- or 40-bit "
                                 "integers on the int8 MFMA with exact int32 sums and fp64 assembly, the rest and every "
                                 "X update as two fp16 terms per entry on the fp16 MFMA (3 passes, fp32 sums); "
                                 "preconditioned gradient: two bf16 terms per fp32 operand on the bf16 MFMA",
                   "fp64_prefix_iters": j64,
                   "fp64_prefix_products": ("fp64 cores" if args.int8_slices == 0 else
                                            "int8 cores, base-256 digits (fp64 cores where the device-side estimate declines)"),
                   "fp16_split_from_iter": jlow, "x_update_on_fp16_cores": xt_lowp,
                   "schedule": "interval-adapted" if args.schedule == 1 else "classical Newton",
                   "workspace_gib": round(run.ws_bytes / 2**30, 1)},
        "breakdown_ms": {"stats_update": round(stats_ms, 3), "inverse_root": round(refresh_ms, 3),
                         "precondition": round(precond_ms, 3), "step_excl_refresh": round(stats_ms + precond_ms, 3),
                         "amortised_step_pf10": round(stats_ms + precond_ms + refresh_ms / 10, 3)},
        "newton_iters": {"min": int(it.min()), "mean": round(float(it.mean()), 2), "max": int(it.max())},
        "not_converged": int((info_h != 0).sum()),
        "wall_ms_timed_region": round(res["wall_ms"], 1),
    }
    out.update(gemm_rooflines(res, args.steps, step_ms, headline=True))
    out["roofline_stats"] = {"bound": "hbm", "achieved": round(stats_bytes / stats_ms / 1e6, 1), "peak": PEAK_HBM,
                             "unit": "GB/s", "frac": round(stats_bytes / stats_ms / 1e6 / PEAK_HBM, 4),
                             "tflops": round(stats_flops / stats_ms / 1e9, 1)}
    # bf16 gradients: U^T = X_R G^T issues 2 bf16 MFMA passes (X_R split), P = X_L U issues 3 (both split)
    out["roofline_precondition"] = {"bound": "mfma", "achieved": round(precond_issued / precond_ms / 1e9, 1),
                                    "peak": PEAK_BF16_MFMA, "unit": "TFLOP/s (bf16 MFMA issued)",
                                    "frac": round(precond_issued / precond_ms / 1e9 / PEAK_BF16_MFMA, 4),
                                    "fp32_equivalent_tflops": round(precond_flops / precond_ms / 1e9, 1),
                                    "gbps": round(precond_bytes / precond_ms / 1e6, 1)}
    log(f"[bench] refresh: {out['refresh_mfma']}")

    out["packed_statistics"] = packed_section(args, torch, ast, run)
    if "cpu" in sections:
        out["cpu_baseline"] = cpu_baseline(run.fsize, run.Ls, run.Rs, shapes, eps_rel)
    if "staleness" in sections:
        out["staleness"] = staleness_section(args, torch, ast, run, stats_ms + precond_ms, refresh_ms)
    del run, Gs, res
    torch.cuda.empty_cache()
    if "soap" in sections:
        out["soap"] = soap_section(args, torch, ast, W, dev)
        torch.cuda.empty_cache()
    if "lowrank" in sections:
        out["lowrank_batch"] = lowrank_section(args, torch, ast, W, dev)
        torch.cuda.empty_cache()
    if "stress" in sections:
        out["stress_4096"] = stress_section(args, torch, ast, W, dev)
    print(json.dumps(out), flush=True)
    return 0


def packed_section(args, torch, ast, run):
    """The same statistics kept in packed lower tiles (the paper's packed triangular SPD storage, Sec. III-E):
    asteria_stats_update reads and writes only the stored tiles, asteria_inverse_root reads them directly."""
    dev = run.Gs[0].device
    shapes = run.shapes
    Lp = [torch.zeros(ast.packed_elems(m), device=dev) for m, n in shapes]
    Rp = [torch.zeros(ast.packed_elems(n), device=dev) for m, n in shapes]
    blocks = ast.Blocks([(G, L, R, 0, 1) for G, L, R in zip(run.Gs, Lp, Rp)])
    factors = ast.Factors([(L, X, 1) for L, X in zip(Lp, run.XLs)] + [(R, X, 1) for R, X in zip(Rp, run.XRs)])
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2 * args.steps + 2)]
    ast.stats_update(blocks, run.beta, ws=run.ws)                     # warm-up, and statistics to take roots of
    for s in range(args.steps):
        ev[2 * s].record()
        ast.stats_update(blocks, run.beta, ws=run.ws)
        ev[2 * s + 1].record()
    ev[-2].record()
    ast.inverse_root(factors, run.eps_rel, relative=True, root=4, opts=run.opts, info=run.info, iters=run.iters, ws=run.ws)
    ev[-1].record()
    torch.cuda.synchronize()
    stats_ms = sum(ev[2 * s].elapsed_time(ev[2 * s + 1]) for s in range(args.steps)) / args.steps
    refresh_ms = ev[-2].elapsed_time(ev[-1])
    stored = sum(4 * (ast.packed_elems(m) + ast.packed_elems(n)) for m, n in shapes)
    full = sum(4 * (m * m + n * n) for m, n in shapes)
    moved = sum(2 * m * n for m, n in shapes) + 2 * stored
    log(f"[bench] packed statistics: stats {stats_ms:.2f} ms ({moved / stats_ms / 1e6:.0f} GB/s), refresh {refresh_ms:.1f} ms, "
        f"{stored / 2**30:.2f} GiB instead of {full / 2**30:.2f} GiB")
    return {"stats_update_ms": round(stats_ms, 3), "inverse_root_ms": round(refresh_ms, 3),
            "statistics_gib": round(stored / 2**30, 3), "statistics_full_storage_gib": round(full / 2**30, 3),
            "roofline_stats": {"bound": "hbm", "achieved": round(moved / stats_ms / 1e6, 1), "peak": PEAK_HBM, "unit": "GB/s",
                               "frac": round(moved / stats_ms / 1e6 / PEAK_HBM, 4), "bytes": moved},
            "not_converged": int((run.info != 0).sum())}


def staleness_section(args, torch, ast, run, step_ms, refresh_ms):
    """The one part of the paper's runtime that applies to a single large-HBM GPU (its Sec. III-D
    staleness barrier, swept in Sec. IV-C over S in {1, 2, 3, 5, 10}): the refresh runs on a second
    stream behind the training steps and its roots are published under a version counter; a step may
    use roots that are at most S refresh periods old and otherwise waits for the refresh in flight.
    Mock loop: `pf` = 10 steps (statistics + preconditioned gradient of every block, the per-step work
    of the method) per refresh period, five periods per setting; reported is the time the steps of one
    period spend waiting for a refresh ("exposed" refresh time), the period's wall time and how many
    refreshes were started in the window (without waiting the steps of a period can finish before its
    refresh does; the next refresh then starts late)."""
    from paper_2605_16184_amd.staleness import RefreshPipeline
    pf, periods = 10, 5
    out = {"pf": pf, "periods_timed": periods, "step_ms": round(step_ms, 3), "refresh_ms": round(refresh_ms, 3),
           "synchronous_period_ms": round(pf * step_ms + refresh_ms, 1), "sweep": []}
    pipe = RefreshPipeline(torch, ast, run, pf=pf)
    for S in (0, 1, 2, 3, 5, 10):
        r = pipe.run(periods, S)
        out["sweep"].append({"S": S, "period_ms": round(r["period_ms"], 1), "refreshes_started": r["refreshes_started"],
                             "exposed_refresh_ms": round(r["exposed_ms"], 1),
                             "max_step_ms": round(r["max_step_ms"], 1), "median_step_ms": round(r["median_step_ms"], 1),
                             "max_version_age_used": r["max_age"], "not_converged": r["not_converged"]})
        log(f"[bench] staleness S={S}: period {r['period_ms']:.1f} ms ({r['refreshes_started']} refreshes started in {periods}), "
            f"exposed refresh {r['exposed_ms']:.1f} ms, longest step "
            f"{r['max_step_ms']:.1f} ms (median {r['median_step_ms']:.1f}), oldest roots used {r['max_age']} periods")
    del pipe
    return out


def lowrank_section(args, torch, ast, W, dev):
    """Batch of 64 independent 1024 x 1024 blocks, bf16 gradients = rank-32 Gaussian factors x 0.01 plus
    N(0, 1e-4^2) noise, fp32 statistics, beta = 0.95, eps = 1e-6 lambda_max: stats + roots + precondition."""
    nb, n = 64, 1024
    shapes = [(n, n)] * nb
    Gs = [W.lowrank_block(n, n, dev, 2, b) for b in range(nb)]
    run = RootRun(torch, ast, Gs, shapes, 0.95, 1e-6, ast.RootOpts(), args.ws_gib)
    steps = max(2, args.steps)
    res = run.timed(steps, 1, "64x1024")
    it = res["iters"]
    r = gemm_rooflines(res, steps, res["step_ms"])
    log(f"[bench] 64x1024 low-rank: stats {res['stats_ms']:.2f} ms, roots {res['refresh_ms']:.1f} ms, precondition {res['precond_ms']:.2f} ms")
    return {"workload": "64 blocks 1024x1024, rank-32 + noise bf16 gradients, eps=1e-6*lambda_max", "blocks": nb, "factors": 2 * nb,
            "stats_update_ms": round(res["stats_ms"], 3), "inverse_root_ms": round(res["refresh_ms"], 3),
            "precondition_ms": round(res["precond_ms"], 3),
            "newton_iters": {"min": int(it.min()), "mean": round(float(it.mean()), 2), "max": int(it.max())},
            "not_converged": int((res["info"] != 0).sum()),
            "precision_plan": {"fp64_prefix_iters": run.plan[0], "fp16_split_from_iter": run.plan[1]},
            "refresh_mfma": r["refresh_mfma"], "gemm_time_share_ms_per_step": r["gemm_time_share_ms_per_step"]}


def stress_section(args, torch, ast, W, dev):
    """Ill-conditioned stress: 8 blocks of 4096 x 4096, bf16 gradients with singular values log-spaced over
    1e0 .. 1e-8, fp32 statistics accumulated in fp64 (eps = 1e-8 lambda_max needs lambda_min > -eps / 2),
    inverse 4th roots and preconditioned gradients; reports the Newton iteration count and the precision plan
    (the accuracy against the oracle is what tests/test_configs_gpu.py grades)."""
    nb, n = 8, 4096
    shapes = [(n, n)] * nb
    Gs = []
    for b in range(nb):
        U, V = W.haar(n, dev, 500 + b, dtype=torch.float64), W.haar(n, dev, 600 + b, dtype=torch.float64)
        Gs.append(((U * W.logspaced_sigma(n, 8.0, dev)) @ V.T).to(torch.bfloat16))
        del U, V
    run = RootRun(torch, ast, Gs, shapes, 0.95, 1e-8, ast.RootOpts(), args.ws_gib, acc=1)
    res = run.timed(2, 1, "8x4096")
    it = res["iters"]
    r = gemm_rooflines(res, 2, res["step_ms"])
    log(f"[bench] 8x4096 stress: stats (fp64 accumulation) {res['stats_ms']:.1f} ms, roots {res['refresh_ms']:.1f} ms, "
        f"precondition {res['precond_ms']:.1f} ms, iterations {it.min()}..{it.max()}")
    return {"workload": "8 blocks 4096x4096, bf16 gradients with singular values log-spaced over 8 decades, "
                        "fp32 statistics (fp64 accumulation), eps=1e-8*lambda_max", "blocks": nb, "factors": 2 * nb,
            "stats_update_fp64_acc_ms": round(res["stats_ms"], 3),
            "stats_update_fp64_tflops": round(2 * nb * sym_gemm_flops(n) / res["stats_ms"] / 1e9, 1),
            "inverse_root_ms": round(res["refresh_ms"], 3), "precondition_ms": round(res["precond_ms"], 3),
            "newton_iters": {"min": int(it.min()), "mean": round(float(it.mean()), 2), "max": int(it.max())},
            "not_converged": int((res["info"] != 0).sum()),
            "precision_plan": {"fp64_prefix_iters": run.plan[0], "fp16_split_from_iter": run.plan[1]},
            "refresh_mfma": r["refresh_mfma"], "gemm_time_share_ms_per_step": r["gemm_time_share_ms_per_step"],
            "roofline_int8_slices": r.get("roofline_int8_slices")}


def soap_section(args, torch, ast, W, dev):
    """SOAP variant on the same model, blocks <= 2048 (318 blocks, 636 factors): three warm
    refreshes from Q = I, then `steps` x (soap_step + stats_update) and one eigenbasis refresh,
    each timed with events on the stream the library launches on."""
    beta, b1, b2, adam_eps = 0.95, 0.9, 0.95, 1e-8
    shapes = W.block_shapes(W.llama_1b_matrices(), 2048)
    if args.max_blocks:
        shapes = shapes[:: max(1, len(shapes) // args.max_blocks)][: args.max_blocks]
    bank = W.TemplateBank(dev, qr_on_host=True)
    bases = [(bank.get(m, b), bank.get(n, b + 3)) for b, (m, n) in enumerate(shapes)]
    nsets = 2                                   # two gradient sets, used alternately
    Gsets = [[W.soap_gradient(U, V, t, dev, b) for b, (U, V) in enumerate(bases)] for t in range(nsets)]
    Ls = [torch.zeros(m, m, device=dev) for m, n in shapes]
    Rs = [torch.zeros(n, n, device=dev) for m, n in shapes]
    QLs = [torch.eye(m, device=dev) for m, n in shapes]
    QRs = [torch.eye(n, device=dev) for m, n in shapes]
    Ms = [torch.zeros(m, n, device=dev) for m, n in shapes]
    Vs = [torch.zeros(m, n, device=dev) for m, n in shapes]
    Ns = [torch.empty(m, n, device=dev) for m, n in shapes]
    blocks = [ast.Blocks(list(zip(G, Ls, Rs))) for G in Gsets]
    # the step reads Q^T along rows: the transposes are kept beside the bases, and every refresh leaves the
    # new ones there (the bases start as the identity, which is its own transpose)
    QLts = [torch.eye(m, device=dev) for m, n in shapes]
    QRts = [torch.eye(n, device=dev) for m, n in shapes]
    qts = QLts + QRts
    sblocks = [ast.SBlocks(list(zip(G, QLs, QRs, Ms, Vs, Ns, QLts, QRts))) for G in Gsets]
    factors = ast.Factors(list(zip(Ls, QLs)) + list(zip(Rs, QRs)))
    fsize = [m for m, n in shapes] + [n for m, n in shapes]
    need = max(ast.soap_refresh_workspace_bytes(factors)[0], ast.soap_step_workspace_bytes(sblocks[0]),
               ast.stats_update_workspace_bytes(blocks[0]))
    ws = torch.empty(int(need), dtype=torch.uint8, device=dev)
    info = torch.zeros(len(factors), dtype=torch.int32, device=dev)
    torch.cuda.synchronize()
    log(f"[bench] soap: {len(shapes)} blocks, {len(factors)} factors, workspace {need / 2**30:.1f} GiB, "
        f"{torch.cuda.memory_allocated() / 2**30:.1f} GiB resident")
    aux = [torch.cuda.Stream() for _ in range(max(1, min(4, args.soap_groups)))]   # groups of factors side by side (default priority)
    for w in range(3):                          # warm the bases from the identity
        ast.stats_update(blocks[w % nsets], beta, ws=ws)
        ast.soap_refresh(factors, info=info, ws=ws, aux_streams=aux, qt=qts, qt_valid=True)
    torch.cuda.synchronize()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(args.steps)]
    for t in range(args.steps):
        ev[t][0].record()
        ast.soap_step(sblocks[t % nsets], b1, b2, adam_eps, t + 1, ws=ws)
        ev[t][1].record()
        ast.stats_update(blocks[t % nsets], beta, ws=ws)
        ev[t][2].record()
    r0, r1, r2, r3 = (torch.cuda.Event(enable_timing=True) for _ in range(4))
    torch.cuda.synchronize()                                # the device is idle: the host time of the call means something
    r0.record()
    t_host = time.time()
    ast.soap_refresh(factors, info=info, ws=ws, aux_streams=aux, qt=qts, qt_valid=True)
    enqueue_ms = 1e3 * (time.time() - t_host)               # the call returns once everything is enqueued
    r1.record()
    torch.cuda.synchronize()
    r2.record()
    ast.soap_refresh(factors, info=info, ws=ws, qt=qts, qt_valid=True)   # the same refresh on the caller's stream alone
    r3.record()
    torch.cuda.synchronize()
    step_ms = sum(e[0].elapsed_time(e[1]) for e in ev) / args.steps
    stats_ms = sum(e[1].elapsed_time(e[2]) for e in ev) / args.steps
    refresh_ms, refresh1_ms = r0.elapsed_time(r1), r2.elapsed_time(r3)
    # sanity of the refreshed bases (fp64 check of two factors, largest first, and of up to six
    # factors that the refresh reported as failed)
    def orth_of(Q):
        q = Q.double()
        return float(torch.linalg.norm(q.T @ q - torch.eye(q.shape[0], device=dev, dtype=torch.float64)) / q.shape[0] ** 0.5)
    allQ = QLs + QRs
    # ... plus the right factor of the first wide block (m < n / 4): its statistic has rank <= 5 m < n
    # after the five updates of this section, the case the refresh handles with a third sweep
    wide = [len(shapes) + b for b, (m, n) in enumerate(shapes) if 4 * m < n][:1]
    orth = max([orth_of(QLs[0]), orth_of(QRs[-1])] + [orth_of(allQ[i]) for i in wide])
    flagged = [i for i, v in enumerate(info.cpu().tolist()) if v != 0]
    orth_flagged = max([orth_of(allQ[i]) for i in flagged[:: max(1, len(flagged) // 6)][:6]], default=0.0)
    if flagged:
        log(f"[bench] soap: {len(flagged)} factors reported failed, sizes {sorted(set(fsize[i] for i in flagged))}, "
            f"orthogonality of a sample of them {orth_flagged:.1e}")
    step_flops = sum(2.0 * (2.0 * m * m * n + 2.0 * m * n * n) for m, n in shapes)
    step_issued = sum((2.0 + 3.0) * 2.0 * m * n * n + (3.0 + 3.0) * 2.0 * m * m * n for m, n in shapes)
    refresh_flops = sum((2.0 + 8.0 / 3.0) * float(n) ** 3 for n in fsize)
    adam_bytes = sum(24.0 * m * n for m, n in shapes)
    log(f"[bench] soap: step {step_ms:.1f} ms + stats {stats_ms:.1f} ms, refresh {refresh_ms:.1f} ms "
        f"({refresh1_ms:.1f} ms on one stream), orthogonality {orth:.1e}, info!=0: {int((info != 0).sum())}")
    return {"workload": "same 1.1B model, blocks <=2048: 318 blocks, 636 factors; shared singular bases, "
                        "+-30% sigma jitter, 10% dense noise; beta1=0.9, beta2=0.95",
            "blocks": len(shapes), "factors": len(factors),
            "soap_step_ms": round(step_ms, 3), "stats_update_ms": round(stats_ms, 3),
            "refresh_ms": round(refresh_ms, 3), "refresh_single_stream_ms": round(refresh1_ms, 3), "refresh_host_enqueue_ms": round(enqueue_ms, 1),
            "amortised_step_pf10": round(step_ms + stats_ms + refresh_ms / 10, 3),
            "soap_step_tflops": round(step_flops / step_ms / 1e9, 1),
            # bf16 gradients: G Q_R issues 2 bf16 MFMA passes, the other three products 3 each (split operands)
            "soap_step_bf16_issued_tflops": round(step_issued / step_ms / 1e9, 1),
            "soap_step_frac_bf16_mfma": round(step_issued / step_ms / 1e9 / PEAK_BF16_MFMA, 4),
            "refresh_dense_tflops": round(refresh_flops / refresh_ms / 1e9, 1),
            "adam_bytes_gb": round(adam_bytes / 1e9, 2),
            "orthogonality_max": max(orth, orth_flagged), "not_ok": int((info != 0).sum())}


def cpu_baseline(fsize, Ls, Rs, shapes, eps_rel):
    """The float64 oracle (cyclic Jacobi + explicit spectral root), one factor per host thread, on
    a bounded sample of the same statistics; extrapolated to the full refresh by n^3."""
    import numpy as np
    import torch
    import oracle

    cores = min(16, os.cpu_count() or 1, int(os.environ.get("OMP_NUM_THREADS", "16")))
    sample = [L for L, (m, n) in zip(Ls, shapes) if m == 512][:cores]
    if len(sample) < cores:
        sample += [R for R, (m, n) in zip(Rs, shapes) if n == 512][: cores - len(sample)]
    if not sample:                      # truncated debug batch: take the smallest factors
        sample = sorted(Ls + Rs, key=lambda t: t.shape[0])[:cores]
    As = [a.detach().to("cpu", torch.float32).double().numpy() for a in sample]
    os.environ["OMP_NUM_THREADS"] = str(cores)
    t = time.time()
    Xs, lmax, status = oracle.inverse_root_batch(As, eps_rel)
    dt = time.time() - t
    work_sample = sum(a.shape[0] ** 3 for a in As)
    work_full = sum(float(n) ** 3 for n in fsize)
    full_ms = 1e3 * dt * work_full / work_sample
    log(f"[bench] oracle: {len(As)} factors n={As[0].shape[0]} on {cores} threads in {dt:.1f} s "
        f"-> extrapolated full refresh {full_ms / 1e3:.0f} s")
    return {"value": round(full_ms, 1), "unit": "ms per full refresh (extrapolated by n^3 from the sample)",
            "cores": cores, "kind": "oracle", "measured_s": round(dt, 2),
            "sample": f"{len(As)} factors of n={As[0].shape[0]} from this workload's statistics, one per thread "
                      f"(cyclic-Jacobi float64 inverse 4th root), status ok: {int((status == 0).sum())}/{len(As)}"}


if __name__ == "__main__":
    sys.exit(main())
