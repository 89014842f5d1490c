#!/usr/bin/env python3
"""Benchmark of the RSA hot path on one MI355X: one step = rsa_forward + rsa_backward
(fused mode) over one batch of synthetic BERT-shaped Q, K, V, dO resident in HBM.

Prints ONE JSON line.  `value` is algorithmic TFLOP/s: 12 * B * Z * A * (visible
query-key pairs) flops per step (4 forward: QK^T, PV; 8 backward: dV, dP, dQ, dK;
recomputation and softmax flops are not credited) over the wall time of the timed
steps.  `roofline` prices the dominant kernel (the fused dK/dV kernel) against
the bf16 dense MFMA peak, launched by its own entry point (`kernel_ms_of`: where rsa_backward
forms dQ and dK, dV in one grid, as for bert_base, `kernel_ms` are those of the kernels one by
one and add up to more than the step); `mfma_executed_tflops` / `mfma_util` count what the matrix
cores actually execute (9 GEMM units for the 6 algorithmic ones: the backward
recomputes the scores in both of its kernels and dP in the dQ kernel);
`cpu_baseline` times the fp64 oracle on the host cores on a bounded sample of the
same workload.  The default workload is long_32k, the largest whole-ring
configuration; the others follow under `other_workloads`, each with its own
`roofline`.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA peak
PEAK_HBM_GBS = 8000.0

# GEMM units (one unit = 2 * B * Z * A * pairs flops) per kernel: credited to the paper's method /
# executed by the kernel.  The dK/dV kernel forms S, dP, dV, dK (S is recomputation), the dQ
# kernel S, dP, dQ (S and dP are), the forward S and P V.
UNITS = {"fwd": (2, 2), "bwd_dkdv": (3, 4), "bwd_dq": (1, 3)}
KERNEL_NAMES = {"fwd": "fused_fwd_kernel", "bwd_dkdv": "fused_bwd_dkdv_kernel", "bwd_dq": "fused_bwd_dq_kernel"}


def measured_traffic(workload, kernel):
    """HBM bytes per launch of `kernel` on `workload`, from the tracked summary of two
    rocprofv3 --pmc runs (FETCH_SIZE, then WRITE_SIZE, each scaled by what the same counter
    reads for a device copy of known size): the line `traffic_bytes_per_launch[<kernel>] = N`
    of profiles/rsa_fused_<workload>_hbm_traffic.txt.  None where no such summary exists."""
    path = os.path.join(ROOT, "profiles", f"rsa_fused_{workload}_hbm_traffic.txt")
    key = f"traffic_bytes_per_launch[{kernel}]"
    try:
        with open(path) as f:
            for line in f:
                if line.startswith(key):
                    return float(line.split("=")[1])
    except OSError:
        pass
    return None


def rooflines(cfg, kernel_ms):
    """Per kernel: algorithmic and executed TFLOP/s against the bf16 dense MFMA peak."""
    unit = 2.0 * cfg.B * cfg.Z * cfg.A * cfg.visible_pairs()
    out = {}
    for k, (alg, exe) in UNITS.items():
        t = kernel_ms[k] * 1e-3
        a, e = alg * unit / t / 1e12, exe * unit / t / 1e12
        out[k] = {"bound": "mfma", "kernel": KERNEL_NAMES[k], "achieved": round(a, 2), "peak": PEAK_BF16_TFLOPS,
                  "unit": "TFLOP/s", "frac": round(a / PEAK_BF16_TFLOPS, 4),
                  "executed": round(e, 2), "executed_frac": round(e / PEAK_BF16_TFLOPS, 4),
                  "traffic": measured_traffic(cfg.name, KERNEL_NAMES[k])}
    return out


def workload_summary(cfg, res):
    """What the line carries for one workload besides its throughput."""
    r = rooflines(cfg, res["kernel_ms"])
    executed = 1.5 * res["tflops"]     # 9 executed GEMM units for 6 algorithmic ones (masked halves of
    return {                           # diagonal tiles, executed under the causal mask, not counted)
        "tflops": round(res["tflops"], 2), "ms_per_step": round(res["ms_per_step"], 4),
        "frac_of_bf16_peak": round(res["tflops"] / PEAK_BF16_TFLOPS, 4),
        "mfma_executed_tflops": round(executed, 2), "mfma_util": round(executed / PEAK_BF16_TFLOPS, 4),
        "kernel_ms": {n: round(v, 4) for n, v in res["kernel_ms"].items()},
        "kernel_ms_of": "step-level entry points, one kernel at a time",
        "roofline": r["bwd_dkdv"], "kernel_rooflines": {k: r[k] for k in ("fwd", "bwd_dq")},
    }


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    # The chip needs on the order of 100 ms of back-to-back launches before its clocks settle:
    # kernel times measured over 20 launches are about 10 % longer than over 1000.  The
    # defaults (set in main) give about 0.2 s of warm-up and 1.5 s of timed steps.
    ap.add_argument("--steps", type=int, default=None)
    ap.add_argument("--warmup", type=int, default=None)
    ap.add_argument("--workload", default="long_32k",
                    choices=["bert_base", "bert_large", "long_32k", "rank15_64k_causal",
                             "causal_ring_32k", "zigzag_rank0_64k_causal", "wide_heads_8k"])
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--all", action="store_true", help="(default) also time the other workloads briefly")
    ap.add_argument("--only", action="store_true", help="time the chosen workload only (no extra legs)")
    ap.add_argument("--legs", default="others,projections,linformer",
                    help="extra legs after the timed region: the other workloads, the projections around RSA, "
                         "the Linformer variant (comma-separated subset)")
    ap.add_argument("--staged", action="store_true",
                    help="also time the staged (two-pass) kernels of one rank: HBM GB/s of the score strip")
    ap.add_argument("--profile-copy", type=int, default=0, metavar="BYTES",
                    help="after the timed steps, run a plain device copy of BYTES three times "
                         "(the known-size kernel that calibrates rocprofv3's FETCH_SIZE / WRITE_SIZE)")
    return ap.parse_args()


def event_ms(fn, iters, torch):
    """Average duration of fn() in ms, HIP events on the current stream."""
    s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    s.record()
    for _ in range(iters):
        fn()
    e.record()
    e.synchronize()
    return s.elapsed_time(e) / iters


def event_stats(fns, iters, torch):
    """Median and minimum over `iters` single passes of every function in fns (run one after the
    other inside each pass), each pass bracketed by its own HIP events: {name: (median, min)} in ms,
    plus "step" for the whole pass."""
    names = list(fns)
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(len(names) + 1)] for _ in range(iters)]
    torch.cuda.synchronize()
    for it in range(iters):
        ev[it][0].record()
        for j, n in enumerate(names):
            fns[n]()
            ev[it][j + 1].record()
    torch.cuda.synchronize()
    out = {}
    for j, n in enumerate(names):
        t = sorted(ev[it][j].elapsed_time(ev[it][j + 1]) for it in range(iters))
        out[n] = (t[len(t) // 2], t[0])
    t = sorted(ev[it][0].elapsed_time(ev[it][-1]) for it in range(iters))
    out["step"] = (t[len(t) // 2], t[0])
    return out


def setup(cfg, torch, rsa, inputs):
    x = inputs.make_inputs(cfg)
    dt = torch.bfloat16
    t = {k: torch.from_numpy(v).to(dt).cuda().contiguous() for k, v in x.items()}
    rb, re = cfg.ranks
    desc = rsa.make_desc(t["K"], cfg.N, causal=cfg.causal, rank_begin=rb, rank_end=re, zigzag=cfg.zigzag)
    buf = dict(
        O=torch.empty_like(t["Q"]), LSE=torch.empty(t["Q"].shape[:3], dtype=torch.float32, device="cuda"),
        dQ=torch.empty_like(t["Q"]), dK=torch.empty_like(t["K"]), dV=torch.empty_like(t["V"]),
        ws=torch.empty(max(rsa.workspace_bytes(desc, True), 16), dtype=torch.uint8, device="cuda"),
        ws_fwd=torch.empty(max(rsa.workspace_bytes(desc, False), 16), dtype=torch.uint8, device="cuda"),
    )
    return x, t, desc, buf


def time_workload(cfg, steps, warmup, torch, rsa, inputs, per_kernel=True, preheat_s=0.3):
    x, t, desc, b = setup(cfg, torch, rsa, inputs)

    def fwd():
        rsa.forward(desc, t["Q"], t["K"], t["V"], O=b["O"], LSE=b["LSE"], ws=b["ws_fwd"])

    def bwd():
        rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], b["O"], b["LSE"],
                     dQ=b["dQ"], dK=b["dK"], dV=b["dV"], ws=b["ws"])

    def step():
        fwd()
        bwd()

    # Untimed preheat before the W warm-up steps: the chip's clocks need some 100 ms of back-to-back
    # launches to settle (kernel times read 10 % longer over the first 20 launches than in steady state).
    t_pre = time.perf_counter()
    while time.perf_counter() - t_pre < preheat_s:
        for _ in range(8):
            step()
        torch.cuda.synchronize()
    for _ in range(warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        step()
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    res = {"ms_per_step": ms, "tflops": cfg.flops() / (ms * 1e-3) / 1e12,
           "tokens_per_s": cfg.B * cfg.Lq / (ms * 1e-3)}
    if per_kernel:
        it = max(3, min(steps, 400))
        for _ in range(min(warmup, 50)):   # keep the clocks up between the two timed regions
            step()
        k = {
            "fwd": event_ms(fwd, it, torch),
            "bwd_preprocess": event_ms(lambda: rsa.bwd_preprocess(desc, t["dO"], b["O"], b["LSE"],
                                                                  b["ws"]),
                                       it, torch),
            "bwd_dkdv": event_ms(lambda: rsa.bwd_dkdv(desc, t["dO"], t["Q"], t["K"], t["V"], b["ws"], b["dK"],
                                                      b["dV"]),
                                 it, torch),
            "bwd_dq": event_ms(lambda: rsa.bwd_dq(desc, t["dO"], t["Q"], t["K"], t["V"], b["ws"], b["dQ"]),
                               it, torch),
        }
        res["kernel_ms"] = k
        st = event_stats({"fwd": fwd, "bwd": bwd}, max(5, min(steps, 200)), torch)
        res["pass_ms"] = {n: {"median": round(v[0], 4), "min": round(v[1], 4)} for n, v in st.items()}
    return res, x


def projections_report(cfg, torch, rsa):
    """The linear maps around RSA (Table 2, rows Q/K/V and Linear) on cfg's rows, H = Z*A:
    forward (2 products) and backward (4 products) timed with HIP events."""
    H = cfg.Z * cfg.A
    rows = cfg.Lq
    g = torch.Generator(device="cuda").manual_seed(0)
    rnd = lambda *shape, s=1.0: (torch.randn(shape, generator=g, device="cuda") * s).to(torch.bfloat16)
    X, dY = rnd(cfg.B, rows, H), rnd(cfg.B, rows, H)
    W, Wo = rnd(H, 3 * H, s=H ** -0.5), rnd(H, H, s=H ** -0.5)
    heads = lambda: rnd(cfg.B, cfg.Z, rows, cfg.A)
    O, dQ, dK, dV = heads(), heads(), heads(), heads()
    Kfull = torch.empty((cfg.B, cfg.Z, cfg.L, cfg.A), dtype=torch.bfloat16, device="cuda")
    rb, re = cfg.ranks
    desc = rsa.make_desc(Kfull, cfg.N, rank_begin=rb, rank_end=re)
    Q, K, V = rsa.qkv_proj(desc, X, W)
    Y = rsa.out_proj(desc, O, Wo)
    ws = torch.empty(max(rsa.proj_workspace_bytes(desc, H), 16), dtype=torch.uint8, device="cuda")
    dO, dWo = rsa.out_proj_bwd(desc, dY, O, Wo, ws=ws)
    dX, dW = rsa.qkv_proj_bwd(desc, dQ, dK, dV, X, W, ws=ws)

    def fwd():
        rsa.qkv_proj(desc, X, W, Q, K, V)
        rsa.out_proj(desc, O, Wo, Y)

    def bwd():
        rsa.out_proj_bwd(desc, dY, O, Wo, dO, dWo, ws)
        rsa.qkv_proj_bwd(desc, dQ, dK, dV, X, W, dX, dW, ws)

    for _ in range(100):
        fwd(); bwd()
    tf, tb = event_ms(fwd, 200, torch), event_ms(bwd, 200, torch)
    M = cfg.B * rows
    f_fwd = 2.0 * M * H * 4 * H            # X W (3H columns) + O Wo
    return {"H": H, "rows": M, "fwd_ms": round(tf, 4), "bwd_ms": round(tb, 4),
            "fwd_tflops": round(f_fwd / (tf * 1e-3) / 1e12, 1),
            "bwd_tflops": round(2 * f_fwd / (tb * 1e-3) / 1e12, 1),
            "frac_of_bf16_peak": round(3 * f_fwd / ((tf + tb) * 1e-3) / 1e12 / PEAK_BF16_TFLOPS, 4)}


def linformer_report(torch, rsa):
    """The Linformer variant (Table 3) at the paper's sequence-length upper bound (section 4.4):
    114688 tokens, batch 4, BERT-Base heads (Z = 12, A = 64), 32 ranks simulated on the one GPU,
    projection dimension 256.  Forward = 2 projections + attention; backward = attention backward +
    2 projection backwards.  Flops: 4*B*Z*L*Kp*A per projection pair and per attention product pair."""
    B, Z, A, L, N, Kp = 4, 12, 64, 114688, 32, 256
    g = torch.Generator(device="cuda").manual_seed(0)
    rnd = lambda *shape, s=1.0: (torch.randn(shape, generator=g, device="cuda") * s).to(torch.bfloat16)
    Q, K, V, dO = (rnd(B, Z, L, A) for _ in range(4))
    E, F = rnd(L, Kp, s=L ** -0.5), rnd(L, Kp, s=L ** -0.5)
    desc = rsa.make_desc(K, N)
    ws = torch.empty(max(rsa.linformer_workspace_bytes(desc, Kp), 16), dtype=torch.uint8, device="cuda")
    Kp_, Vp_ = rsa.linformer_project(desc, K, E, ws=ws), rsa.linformer_project(desc, V, F, ws=ws)
    O, LSE = rsa.linformer_forward(desc, Q, Kp_, Vp_)
    dQ, dKp, dVp = rsa.linformer_backward(desc, dO, Q, Kp_, Vp_, O, LSE, ws=ws)
    dK, dE = rsa.linformer_project_bwd(desc, dKp, K, E)
    dV, dF = rsa.linformer_project_bwd(desc, dVp, V, F)

    def fwd():
        rsa.linformer_project(desc, K, E, Kp_, ws)
        rsa.linformer_project(desc, V, F, Vp_, ws)
        rsa.linformer_forward(desc, Q, Kp_, Vp_, O, LSE)

    def bwd():
        rsa.linformer_backward(desc, dO, Q, Kp_, Vp_, O, LSE, dQ, dKp, dVp, ws)
        rsa.linformer_project_bwd(desc, dKp, K, E, dK, dE)
        rsa.linformer_project_bwd(desc, dVp, V, F, dV, dF)

    for _ in range(10):
        fwd(); bwd()
    tf, tb = event_ms(fwd, 20, torch), event_ms(bwd, 20, torch)
    pair = 4.0 * B * Z * L * Kp * A            # two products of 2*B*Z*L*Kp*A flops
    flops_f, flops_b = 2 * pair, 4 * pair      # fwd: projections + QK^T, PV; bwd: twice that
    return {"B": B, "Z": Z, "L": L, "N": N, "Kp": Kp, "fwd_ms": round(tf, 3), "bwd_ms": round(tb, 3),
            "tflops": round((flops_f + flops_b) / ((tf + tb) * 1e-3) / 1e12, 1),
            "tokens_per_s": round(B * L / ((tf + tb) * 1e-3), 1),
            "hbm_gb_resident": round(torch.cuda.max_memory_allocated() / 1e9, 2)}


def staged_report(cfg, torch, rsa, inputs):
    """The paper's two-pass layout for one simulated rank (rank 0): time every ring step
    kernel with HIP events and price the memory-bound ones against HBM."""
    x = inputs.make_inputs(cfg)
    t = {k: torch.from_numpy(v).to(torch.bfloat16).cuda().contiguous() for k, v in x.items()}
    desc = rsa.make_desc(t["K"], cfg.N, causal=cfg.causal, mode=rsa.MODE_STAGED)
    n, c, L, N, heads = 0, cfg.c, cfg.L, cfg.N, cfg.B * cfg.Z
    dev = t["K"].device
    S = torch.empty((cfg.B, cfg.Z, c, L), dtype=torch.float32, device=dev)
    P = torch.empty((cfg.B, cfg.Z, c, L), dtype=torch.bfloat16, device=dev)
    dS = torch.empty_like(P)
    LSE = torch.empty((cfg.B, cfg.Z, cfg.L), dtype=torch.float32, device=dev)
    D = torch.zeros_like(LSE)
    Oacc = torch.empty((cfg.B, cfg.Z, c, cfg.A), dtype=torch.float32, device=dev)
    for j in range(N):
        rsa.qk_step(desc, n, j, t["Q"], t["K"], S)
    scores = heads * c * L
    ms = {
        "qk_step": event_ms(lambda: rsa.qk_step(desc, n, 1 % N, t["Q"], t["K"], S), 10, torch),
        "row_softmax": event_ms(lambda: rsa.row_softmax(desc, n, S, P, LSE), 10, torch),
        "av_step": event_ms(lambda: rsa.av_step(desc, n, 1 % N, P, t["V"], Oacc, 0), 10, torch),
        "softmax_bwd": event_ms(lambda: rsa.softmax_bwd(desc, n, P, S, D, dS), 10, torch),
    }
    # the whole ring in this layout: every rank's two passes, forward and backward
    del S, P, dS, Oacc
    O = torch.empty_like(t["Q"])
    dQ, dK, dV = torch.empty_like(t["Q"]), torch.empty_like(t["K"]), torch.empty_like(t["V"])
    wf = torch.empty(max(rsa.workspace_bytes(desc, False), 16), dtype=torch.uint8, device=dev)
    wb = torch.empty(max(rsa.workspace_bytes(desc, True), 16), dtype=torch.uint8, device=dev)
    ms["ring_forward"] = event_ms(lambda: rsa.forward(desc, t["Q"], t["K"], t["V"], O=O, LSE=LSE, ws=wf), 3, torch)
    ms["ring_backward"] = event_ms(lambda: rsa.backward(desc, t["dO"], t["Q"], t["K"], t["V"], O, LSE, dQ=dQ,
                                                        dK=dK, dV=dV, ws=wb), 3, torch)
    gbs = lambda nbytes, m: nbytes / (m * 1e-3) / 1e9
    # algorithmic bytes: softmax reads 4 B and writes 2 B per score; softmax backward reads
    # P (2 B) and dP (4 B) and writes dS (2 B); a qk step writes 4 B per score of its block
    return {
        "rank": n, "scores_per_rank": scores, "kernel_ms": {k: round(v, 4) for k, v in ms.items()},
        "row_softmax_GBps": round(gbs(6 * scores, ms["row_softmax"]), 1),
        "softmax_bwd_GBps": round(gbs(8 * scores, ms["softmax_bwd"]), 1),
        "qk_step_write_GBps": round(gbs(4 * scores / N, ms["qk_step"]), 1),
        "hbm_peak_GBps": PEAK_HBM_GBS,
        "strip_bytes_forward_all_ranks": (4 + 4 + 2 + 2) * scores * N,
        "ring_tflops": round(cfg.flops() / ((ms["ring_forward"] + ms["ring_backward"]) * 1e-3) / 1e12, 1),
    }


def cpu_baseline(cfg, x, inputs):
    """The fp64 oracle, as it stands, on a bounded head sample of the same workload."""
    import numpy as np
    import oracle
    heads_total = cfg.B * cfg.Z
    per_head = 18.0 * cfg.A * cfg.visible_pairs()        # fp64 flops the oracle executes per head
    heads = int(max(1, min(heads_total, round(2.5e12 / per_head))))   # about 10-30 s of host work
    sel = lambda a: np.ascontiguousarray(
        a.reshape(heads_total, a.shape[2], a.shape[3])[:heads][None].astype(np.float64))
    Q, K, V, dO = (sel(x[k]) for k in ("Q", "K", "V", "dO"))
    dt = 0.0
    for r0, tok0, n in cfg.segments():   # one oracle call per run of consecutive tokens
        Qs, dOs = (np.ascontiguousarray(a[:, :, r0:r0 + n]) for a in (Q, dO))
        t0 = time.perf_counter()
        oracle.forward(Qs, K, V, q0=tok0, causal=cfg.causal)
        oracle.backward(Qs, K, V, dOs, q0=tok0, causal=cfg.causal)
        dt += time.perf_counter() - t0
    flops = 12.0 * heads * cfg.A * cfg.visible_pairs()
    return {"value": flops / dt / 1e12, "unit": "TFLOP/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"first {heads} of {heads_total} (batch, head) pairs of {cfg.name}, fwd+bwd, "
                      f"fp64, {dt:.1f} s"}


def main():
    a = parse()
    if a.gpus != 1:
        print("bench.py: this build runs on one GPU only; the ring's ranks are simulated as chunk "
              "iterations on that GPU (--gpus must be 1)", file=sys.stderr)
        return 2
    import torch
    from paper_2105_13120_amd import inputs, rsa
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 2
    rsa.lib()   # fails loudly if the HIP library is not built
    cfg = inputs.CONFIGS[a.workload]
    # default step count: about as many flops as 2000 steps of bert_large
    scale = inputs.CONFIGS["bert_large"].flops() / cfg.flops()
    if a.steps is None:
        a.steps = int(min(5000, max(20, round(2000 * scale))))
    if a.warmup is None:
        a.warmup = int(min(1000, max(5, round(300 * scale))))
    res, x = time_workload(cfg, a.steps, a.warmup, torch, rsa, inputs)
    summ = workload_summary(cfg, res)
    out = {
        "metric": "rsa_fwd_bwd_tflops", "value": summ["tflops"], "unit": "TFLOP/s",
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup, "ms_per_step": summ["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": cfg.name, "B": cfg.B, "Z": cfg.Z, "L": cfg.L, "A": cfg.A, "N": cfg.N,
                   "chunk": cfg.c, "causal": cfg.causal, "ranks": list(cfg.ranks), "mode": "fused",
                   "ownership": "zigzag" if cfg.zigzag else "contiguous",
                   "why": "long_32k is the largest configuration of the five that runs the whole ring on one GPU; "
                          "bert_large (the smallest that carries the 50 %-of-peak target) and the rest are under "
                          "other_workloads" if cfg.name == "long_32k" else "chosen with --workload"},
        "frac_of_bf16_peak": summ["frac_of_bf16_peak"],
        "mfma_executed_tflops": summ["mfma_executed_tflops"], "mfma_util": summ["mfma_util"],
        "tokens_per_s": round(res["tokens_per_s"], 1),
        "kernel_ms": summ["kernel_ms"],
        "pass_ms": res["pass_ms"],
        "roofline": summ["roofline"], "kernel_rooflines": summ["kernel_rooflines"],
    }
    legs = set() if a.only else set(a.legs.split(","))
    if "others" in legs:
        other = {}
        for name in ("bert_base", "bert_large", "long_32k", "rank15_64k_causal", "causal_ring_32k",
                     "zigzag_rank0_64k_causal", "wide_heads_8k"):
            if name == cfg.name:
                continue
            c2 = inputs.CONFIGS[name]
            s2 = inputs.CONFIGS["bert_large"].flops() / c2.flops()
            r2, _ = time_workload(c2, int(min(2000, max(10, round(500 * s2)))),
                                  int(min(300, max(3, round(100 * s2)))), torch, rsa, inputs, preheat_s=0.1)
            other[name] = workload_summary(c2, r2)
        out["other_workloads"] = other
    if "projections" in legs:
        out["projections"] = projections_report(inputs.CONFIGS["bert_large"], torch, rsa)
    if "linformer" in legs:
        out["linformer_114k"] = linformer_report(torch, rsa)
    if a.staged:
        out["staged"] = staged_report(cfg, torch, rsa, inputs)
    if a.profile_copy > 0:
        src = torch.empty(a.profile_copy, dtype=torch.uint8, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        out["profile_copy_bytes"] = a.profile_copy
    if not a.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(cfg, x, inputs)
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
