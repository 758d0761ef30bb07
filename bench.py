#!/usr/bin/env python3
"""Benchmark of the DTS-Gate MoE layer on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--config gpt] [--no-cpu-baseline]

A "step" is one forward + backward pass of the whole layer (gate, dispatch, expert FFNs, combine and
every backward step) over one batch of T synthetic tokens, inputs already resident in HBM.  Successive
steps walk the config's dense-to-sparse temperature sweep (tau 2.0 -> 0.3), so K steps cover each
temperature K / len(sweep) times.  Prints ONE JSON line.

The metric is MoE-layer tokens/s forward+backward on the GPT-shaped layer (d=768, E=16, T=8192), with
the roofline fraction of the dominant kernel (bf16 MFMA) measured live with HIP events, and the CPU oracle
timed on the host cores on the same workload as a baseline.

After the timed region the same process measures, each labelled in the JSON line: forward and backward
separately at every temperature (median and minimum over repeats), one supplementary point at threshold 0
(every expert selected for every token, P = T*E: the dense limit), a per-kernel event table, and the layer
against the smaller of its two rooflines (bf16 MFMA time of its flops, HBM time of its algorithmic bytes).
"""
from __future__ import annotations

import argparse
import json
import os
import re
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

PEAK_BF16_MFMA_TFLOPS = 2500.0     # MI355X dense bf16
PEAK_FP32_TFLOPS = 157.3
PEAK_HBM_GBS = 8000.0

# the dominant kernel as rocprofv3 names it (the merged weight-gradient launch)
DOMINANT_PROFILE_NAME = "grouped_gemm_bf16<2, 4,"


def _gemm_kernels():
    # expert-FFN GEMM launches and how many 2*P*d*F-flop contractions each carries
    # (ffn_bwd_dw2 is the merged dW2 + dW1 launch; ffn_bwd_db is dO's column sums where they have a launch of their own)
    return {"ffn_gemm1": 1, "ffn_gemm2": 1, "ffn_bwd_dh": 1, "ffn_bwd_dx": 1, "ffn_bwd_dw2": 2}


def profiled_traffic(config):
    """HBM bytes per launch of the dominant kernel, read from the two rocprofv3 --pmc summaries kept under
    profiles/ (FETCH_SIZE and WRITE_SIZE in KiB per dispatch, each scaled by what the counter reads for a plain
    copy of known size; both facts are lines of those files).  None when no summary of this config exists."""
    total = 0.0
    for counter in ("fetch_size", "write_size"):
        path = os.path.join(ROOT, "profiles", f"layer_{config}_pmc_{counter}.txt")
        if not os.path.exists(path):
            return None
        kib = scale = None
        for line in open(path):
            if line.startswith(DOMINANT_PROFILE_NAME) or (not line.startswith("#") and DOMINANT_PROFILE_NAME in line):
                kib = float(line.split()[-1])
            m = re.search(r"true KiB = counter x ([0-9.]+)", line)
            if m:
                scale = float(m.group(1))
        if kib is None or scale is None:
            return None
        total += kib * scale * 1024.0
    return int(total)


def cpu_baseline(cfg, inp, n_tokens, taus, top1=False):
    """The oracle as it stands, timed on the host cores on the first n_tokens tokens over the sweep."""
    import numpy as np
    from oracle import evomoe_oracle as orc
    try:
        from threadpoolctl import threadpool_info
        cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
    except Exception:
        cores = os.cpu_count() or 1
    x, noise, dy = inp.x[:n_tokens], inp.noise[:n_tokens], inp.dy[:n_tokens]
    t0 = time.perf_counter()
    pairs = 0
    for tau in taus:
        override = orc.top1_gate(x, inp.Wg, inp.bg, noise, tau).mask if top1 else None
        fwd = orc.moe_layer_forward(x, inp.Wg, inp.bg, noise, tau, cfg.threshold, inp.W1, inp.b1,
                                    inp.W2, inp.b2, cfg.act, mask_override=override)
        orc.moe_layer_backward(fwd, dy, x, inp.Wg, tau, inp.W1, inp.W2, cfg.act)
        if top1:
            orc.balance_loss(fwd.gate, 0.1)
        pairs += int(fwd.disp.expert_offsets[-1])
    dt = time.perf_counter() - t0
    what = "all" if n_tokens == cfg.T else "the first"
    return {"value": n_tokens * len(taus) / dt, "unit": "tokens/s", "cores": int(cores), "kind": "oracle",
            "sample": f"{what} {n_tokens} tokens of the workload, fwd+bwd at each of the {len(taus)} sweep "
                      f"temperatures ({pairs} pairs, {dt:.1f} s, float64 numpy)"}


def layer_bytes(cfg, P):
    """Algorithmic HBM bytes of one forward + backward pass at P selected pairs: every operand of every step
    read once and every result written once per step that uses it (weights: four reads and two writes)."""
    T, d, E, F = cfg.T, cfg.d, cfg.E, cfg.F
    sz = 2 if cfg.dtype == "bf16" else 4
    gemm = (6 * P * d + 8 * P * F + 6 * E * d * F) * sz
    gate = T * (d * sz + E * 8 + 12) + T * 12 + P * 16                      # gate + dispatch
    stream = (P * d * sz + T * d * sz) * 2 + (2 * P * d * sz + T * d * sz)  # combine, dispatch bwd, combine bwd
    gate_bwd = T * d * sz * 3 + T * E * 12
    return gemm + gate + stream + gate_bwd


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=60)
    ap.add_argument("--warmup", type=int, default=12)
    ap.add_argument("--config", default="gpt")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--mode", choices=("sweep", "top1"), default="sweep",
                    help="sweep: the dense-to-sparse temperature sweep with the threshold gate (headline metric); "
                         "top1: the steady state after the sweep -- Top-1 gate at the final temperature, P = T, "
                         "with the balance loss (alpha = 0.1) in the backward")
    ap.add_argument("--recompute", action="store_true",
                    help="backward recomputes the expert activations instead of reading the forward's")
    ap.add_argument("--cpu-tokens", type=int, default=0, help="tokens of the oracle baseline (0 = all of them)")
    ap.add_argument("--copy-probe", action="store_true",
                    help="after the timed region, run a plain elementwise kernel over 512 MiB three times "
                         "(known traffic each way, to calibrate rocprofv3's FETCH_SIZE / WRITE_SIZE)")
    ap.add_argument("--no-kernel-table", action="store_true",
                    help="skip the passes after the timed region (per-temperature forward/backward times, dense "
                         "limit, per-kernel events)")
    ap.add_argument("--no-hint", action="store_true", help="do not announce the pair count before each step")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build is single-GPU by design (all experts resident, no collectives); "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2112_14397_amd import binding as B
    import synth_inputs as synth

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    cfg = synth.CONFIGS[args.config]
    inp = synth.make_layer_inputs(cfg)
    dt = B.torch_dtype(cfg.dtype)
    dev = lambda a, t=None: None if a is None else (torch.from_numpy(np.ascontiguousarray(a)).cuda().to(t) if t
                                                    else torch.from_numpy(np.ascontiguousarray(a)).cuda())
    x, noise, dy = dev(inp.x, dt), dev(inp.noise), dev(inp.dy, dt)
    params = B.LayerParams(Wg=dev(inp.Wg), bg=dev(inp.bg), W1=dev(inp.W1, dt), b1=dev(inp.b1),
                           W2=dev(inp.W2, dt), b2=dev(inp.b2))
    ctx = B.Context()
    taus = list(cfg.taus)
    top1 = args.mode == "top1"
    if top1:
        taus = [taus[-1]]
    alpha = 0.1 if top1 else None

    # size the per-pair buffers from the sweep's largest P (one untimed gate+dispatch per temperature)
    probe_shape = B.make_shape(cfg.T, cfg.d, cfg.E, 8, cfg.dtype, cfg.act, cfg.T * cfg.E)
    pb = B.LayerBuffers(probe_shape, backward=False)
    P_of = {}
    for tau in taus:
        if top1:
            B.evomoe_dts_gate_top1(ctx, probe_shape, x, params.Wg, params.bg, noise, tau, pb.gprime, None,
                                   pb.mask_bits, pb.counts, pb.k)
        else:
            B.evomoe_dts_gate(ctx, probe_shape, x, params.Wg, params.bg, noise, tau, cfg.threshold, pb.gprime, None,
                              pb.mask_bits, pb.counts, pb.k)
        B.evomoe_dispatch(ctx, probe_shape, pb.mask_bits, pb.gprime, pb.expert_offsets, pb.pair_token,
                          pb.pair_gate, pb.tok_off, pb.tok_rows, pb.num_pairs)
        P_of[tau] = B.evomoe_num_pairs(ctx, pb.num_pairs)
    del pb
    P_cap = int(max(P_of.values()) * 1.02) + 256
    shape = B.make_shape(cfg.T, cfg.d, cfg.E, cfg.F, cfg.dtype, cfg.act, P_cap)
    buf = B.LayerBuffers(shape, backward=True, recompute=args.recompute)

    # A trainer knows the previous iteration's pair count (evomoe_num_pairs) and the schedule moves it slowly:
    # it is announced before every step so that the expert GEMMs pick their tile shapes for it, not for P_cap.
    def hint(tau, P=None):
        if not args.no_hint:
            B.evomoe_hint_pairs(ctx, P_of[tau] if P is None else P)

    def fwd(tau, c=cfg.threshold, b=buf):
        B.layer_forward(ctx, b, params, x, noise, tau, c, write_gate_w=False, top1=top1)

    def bwd(tau, b=buf):
        B.layer_backward(ctx, b, params, x, dy, tau, balance_alpha=alpha, recompute=args.recompute)

    def step(tau):
        hint(tau)
        fwd(tau)
        bwd(tau)

    for i in range(args.warmup):
        step(taus[i % len(taus)])
    torch.cuda.synchronize()

    # the longest launch of a step: the merged weight-gradient GEMM (dW2 and dW1 in one persistent grid)
    dominant = "ffn_bwd_dw2"
    B.evomoe_profile_select(ctx, dominant)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        step(taus[i % len(taus)])
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    prof = B.evomoe_profile_read(ctx)
    B.evomoe_profile_select(ctx, None)

    ms_per_step = elapsed * 1e3 / args.steps
    tokens_per_s = cfg.T * args.steps / elapsed
    flops_per_pair_gemm = 2.0 * cfg.d * cfg.F
    P_steps = [P_of[taus[i % len(taus)]] for i in range(args.steps)]
    dom_ms, dom_n = prof.get(dominant, (0.0, 0))
    dom_flops = _gemm_kernels()[dominant] * sum(P_steps) * flops_per_pair_gemm
    achieved = dom_flops / (dom_ms * 1e-3) / 1e12 if dom_ms > 0 else 0.0
    roofline = {"bound": "mfma", "kernel": dominant + " (grouped_gemm_bf16<2, 4, ...>: dW2 and dW1)",
                "achieved": achieved, "peak": PEAK_BF16_MFMA_TFLOPS,
                "unit": "TFLOP/s", "frac": achieved / PEAK_BF16_MFMA_TFLOPS,
                "traffic": None if (top1 or args.recompute) else profiled_traffic(args.config),
                "avg_launch_us": dom_ms * 1e3 / max(dom_n, 1), "launches": dom_n,
                "flops_per_launch": "2 GEMMs x 2*P*d*F, P = pairs at the step's temperature "
                                    "(sweep average %.0f)" % (sum(P_steps) / len(P_steps))}

    # the whole layer against the smaller of its two rooflines
    Pavg = sum(P_steps) / len(P_steps)
    t_mfma = 6.0 * flops_per_pair_gemm * Pavg / (PEAK_BF16_MFMA_TFLOPS * 1e12)
    t_hbm = layer_bytes(cfg, Pavg) / (PEAK_HBM_GBS * 1e9)
    layer_roofline = {"mfma_us": t_mfma * 1e6, "hbm_us": t_hbm * 1e6, "bound": "hbm" if t_hbm > t_mfma else "mfma",
                      "frac": max(t_mfma, t_hbm) / (ms_per_step * 1e-3),
                      "note": "time the layer's flops need at the bf16 MFMA peak and its algorithmic bytes at the HBM "
                              "peak; frac = the larger of the two / measured step time"}

    out = {
        "metric": f"MoE-layer tokens/s fwd+bwd (d={cfg.d},E={cfg.E},T={cfg.T}) " + ("vs tau" if not top1 else
                                                                                          "Top-1 steady state"),
        "value": tokens_per_s, "unit": "tokens/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": cfg.dtype, "data": "synthetic",
        "config": {"workload": f"{cfg.name}: T={cfg.T} d={cfg.d} E={cfg.E} F={cfg.F} {cfg.act} "
                               + (f"c={cfg.threshold}, tau sweep {[round(t, 3) for t in taus]} (one tau per step, cyclic)"
                                  if not top1 else f"Top-1 gate at tau={taus[0]:.3f}, balance loss alpha=0.1")
                               + (", backward recomputes H and A" if args.recompute else ""),
                   "pairs_per_tau": {f"{t:.3f}": P_of[t] for t in taus}, "P_cap": P_cap,
                   "pair_hint": not args.no_hint},
        "layer_tflops": 6.0 * flops_per_pair_gemm * sum(P_steps) / elapsed / 1e12,
        "roofline": roofline,
        "layer_roofline": layer_roofline,
    }

    def timed_fwd_bwd(tau, reps, c=cfg.threshold, b=buf):
        """Forward and backward timed separately with events on the library's stream; (fwd ms, bwd ms) lists."""
        ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(reps)]
        for e0, e1, e2 in ev:
            e0.record()
            fwd(tau, c, b)
            e1.record()
            bwd(tau, b)
            e2.record()
        torch.cuda.synchronize()
        return [e0.elapsed_time(e1) for e0, e1, _ in ev], [e1.elapsed_time(e2) for _, e1, e2 in ev]

    def summarize(tau, P, f, g):
        tot = [a + b for a, b in zip(f, g)]
        med = statistics.median(tot)
        return {"tau": round(tau, 3), "pairs": P,
                "fwd_ms": {"median": statistics.median(f), "min": min(f)},
                "bwd_ms": {"median": statistics.median(g), "min": min(g)},
                "ms": med, "ms_min": min(tot), "tokens_per_s": cfg.T / med * 1e3,
                "tflops": 6.0 * flops_per_pair_gemm * P / med / 1e9}

    if not args.no_kernel_table:
        # per-temperature throughput: forward and backward timed separately, median and minimum of 20 repeats
        per_tau = []
        for tau in taus:
            hint(tau)
            for _ in range(5):
                fwd(tau); bwd(tau)
            f, g = timed_fwd_bwd(tau, 20)
            per_tau.append(summarize(tau, P_of[tau], f, g))
        out["per_tau"] = per_tau

        if not top1 and not args.recompute:
            # supplementary: the dense limit -- threshold 0, every expert selected for every token (P = T*E)
            P_dense = cfg.T * cfg.E
            dshape = B.make_shape(cfg.T, cfg.d, cfg.E, cfg.F, cfg.dtype, cfg.act, P_dense)
            dbuf = B.LayerBuffers(dshape, backward=True)
            hint(taus[0], P_dense)
            for _ in range(3):
                fwd(taus[0], 0.0, dbuf); bwd(taus[0], dbuf)
            assert B.evomoe_num_pairs(ctx, dbuf.num_pairs) == P_dense
            f, g = timed_fwd_bwd(taus[0], 10, 0.0, dbuf)
            ent = summarize(taus[0], P_dense, f, g)
            ent["note"] = "supplementary: threshold 0 (all experts selected for every token), not part of the sweep"
            out["dense_limit"] = ent
            del dbuf
            torch.cuda.empty_cache()

    if args.copy_probe:
        # a plain elementwise kernel of known traffic: reads 512 MiB, writes 512 MiB (shows up in a kernel
        # trace as torch's bitwise_not elementwise kernel, three dispatches)
        src = torch.ones(128 * 1024 * 1024, dtype=torch.int32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            torch.bitwise_not(src, out=dst)
        torch.cuda.synchronize()
        out["copy_probe_bytes"] = int(src.numel() * 4)

    if not args.no_kernel_table:    # per-kernel event timings of three more sweeps (outside the timed region)
        B.evomoe_profile_select(ctx, "all")
        for i in range(len(taus) * 3):
            step(taus[i % len(taus)])
        allp = B.evomoe_profile_read(ctx)
        B.evomoe_profile_select(ctx, None)
        Psum = sum(P_of[t] for t in taus) * 3
        Pavg = Psum / (3 * len(taus))
        T, d, E, F = cfg.T, cfg.d, cfg.E, cfg.F
        sz = 2 if cfg.dtype == "bf16" else 4
        # algorithmic HBM bytes per launch of the streaming kernels (sweep-average pair count)
        stream_bytes = {
            "gate": T * (d * sz + E * 8 + 12),
            "dispatch_hist": T * 8, "dispatch_scatter": T * 12 + Pavg * 16,
            "combine": Pavg * d * sz + T * d * sz + Pavg * 8,
            "combine_bwd": 2 * Pavg * d * sz + T * d * sz + Pavg * 12,
            # (bf16 layer) the column sums of dO; both types take the bias gradients' other sums inside the GEMM launches
            "ffn_bwd_db": Pavg * d * sz,
            "dispatch_bwd": Pavg * d * sz + T * d * sz,
            "gate_bwd_dz": T * E * 8 + Pavg * 8 + T * 12,
            "gate_bwd_main": T * d * sz * 3 + T * E * 4,
        }
        ks = {}
        for name, (ms, n) in allp.items():
            ent = {"avg_us": ms * 1e3 / n, "launches": n}
            if name in _gemm_kernels():
                ent["tflops"] = _gemm_kernels()[name] * Psum * flops_per_pair_gemm / (ms * 1e-3) / 1e12
                ent["mfma_frac"] = ent["tflops"] / PEAK_BF16_MFMA_TFLOPS
            if name in stream_bytes:
                ent["hbm_gbs"] = stream_bytes[name] / (ms * 1e-3 / n) / 1e9
                ent["hbm_frac"] = ent["hbm_gbs"] / PEAK_HBM_GBS
            ks[name] = ent
        out["kernels"] = ks

    if not args.no_cpu_baseline:
        n_tok = cfg.T if args.cpu_tokens <= 0 else min(args.cpu_tokens, cfg.T)
        if args.cpu_tokens <= 0 and args.config in ("mt", "large", "roberta"):
            n_tok = min(cfg.T, 2048)        # the larger layers: a bounded sample
        out["cpu_baseline"] = cpu_baseline(cfg, inp, n_tok, taus, top1=top1)
    else:
        out["cpu_baseline"] = None
    print(json.dumps(out))


if __name__ == "__main__":
    main()
