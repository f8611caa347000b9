#!/usr/bin/env python3
"""Benchmark of the TNT memory layer (forward + backward) on one MI355X.

A step is one tnt_mem_fwd (saving the chunk-entry states) followed by one
tnt_mem_bwd on the same synthetic batch, i.e. every kernel of the hot path.
Default workload: batch 4, 8 heads, head dim 64, sequence 8192, MLP 64-256-64
(SiLU), global chunk 2048, one local memory with chunk 64 and shard 2048, bf16
inputs (seeded synthetic data; no dataset).

Prints one JSON line with the throughput (tokens/s of fwd+bwd), the roofline
position of the dominant kernel (algorithmic MFMA FLOPs per launch over its
HIP-event launch time measured inside the timed region) and the fp64 CPU
oracle's throughput on a bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16 = 2.5e15      # MI355X dense bf16 MFMA, FLOP/s
PEAK_FP32 = 157.3e12    # MI355X fp32, FLOP/s
PEAK_HBM = 8.0e12       # MI355X HBM3E, bytes/s
METRIC = "memory-layer fwd+bwd tokens/sec at seq 8192; % MFMA bf16 peak (rocprof)"
# the paper's own efficiency figures (Table 1 and the efficiency discussion of
# Sec. 5), quoted as context: whole-model results on other hardware
PAPER_CONTEXT = {
    "time_to_loss": "TNT with local chunk 64 reaches the target loss 17.37x sooner than the "
                    "Titans baseline at chunk 8 (1.12 h vs 19.48 h, Table 1)",
    "step_time": "one 32K-token training step 5.1x faster than Titans at equal chunk 16",
    "hardware": "TPUv5 pod, JAX",
    "note": "context only: whole-model training on other hardware, not this layer's metric",
}


# ----------------------------------------------------------------------------
# algorithmic FLOPs (GEMM work the method needs, per token and head)
# ----------------------------------------------------------------------------
def local_fwd_flops(d, h, C, qk=True):
    # chunk gradients 6dh, dual-form retrieval 8dh + 4C(d+h), state carry 8dh,
    # Q-K projection 4d^2 + 4Cd
    return 22 * d * h + 4 * C * (d + h) + ((4 * d * d + 4 * C * d) if qk else 0)


def local_bwd_flops(d, h, C, qk=True):
    # adjoints of retrieval, carry and inner gradient 44dh + 8Ch + 8Cd,
    # of the Q-K projection 8Cd + 6d^2
    return 44 * d * h + 8 * C * h + 8 * C * d + ((8 * C * d + 6 * d * d) if qk else 0)


def global_fwd_flops(d, h):
    return 18 * d * h     # chunk gradients 6dh, retrieval 4dh, carry 8dh


def global_fwd_step_flops(cfg):
    """The global forward's FLOPs per step: the last chunk's carry and its
    chunk gradients feed only the final state, which the step does not ask for."""
    tok = cfg.B * cfg.H * cfg.L
    return global_fwd_flops(cfg.d, cfg.hid) * tok - 14 * cfg.d * cfg.hid * cfg.B * cfg.H * cfg.C_G


def global_bwd_flops(d, h):
    return 36 * d * h


def step_flops(cfg):
    tok = cfg.B * cfg.H * cfg.L
    f = 0
    if cfg.has_global:
        f += global_fwd_step_flops(cfg) + global_bwd_flops(cfg.d, cfg.hid) * tok
    for (C, _) in cfg.locals_:
        f += (local_fwd_flops(cfg.d, cfg.hid, C, cfg.qk_proj) +
              local_bwd_flops(cfg.d, cfg.hid, C, cfg.qk_proj)) * tok
    return f


def hbm_bytes(cfg, name):
    """Algorithmic HBM bytes of one launch of the gate scan or of one global
    state-carry step (None for other labels).

    global_scan (one per pass): reads the three gates (fp32) of every token of
    every chain and writes six fp32 coefficients per token, plus four per chunk.
    global_carry (one forward chunk): reads the chunk's carry operands D1^T, Hk^T
    (C x hid each) and the four coefficient-scaled K^T, R^T (C x d each) in the
    compute type, reads the entry state (V1, S1, V2, S2: 4 hid d fp32), writes
    the exit state and the next chunk's compute-type copies of V1, V2 (as they
    are and transposed: 4 hid d elements).  global_bwd_carry (one backward chunk): reads the ten
    operands of the entry-adjoint products (Zkbar, Zqbar, Gbar, Hk, Hq: C x hid;
    K, Q, R, Ykbar, dO: C x d) in the compute type, reads the state and the exit
    adjoint, writes the entry adjoint (each 4 hid d fp32)."""
    chains = cfg.B * cfg.H
    d, h, C, L = cfg.d, cfg.hid, cfg.C_G, cfg.L
    cts = 2 if cfg.dtype == 1 else 4
    st = 4 * h * d * 4
    if name == "global_scan":
        return chains * (L * (3 * 4 + 6 * 4) + (L // C) * 16)
    if name == "global_carry":
        return chains * ((2 * h + 4 * d) * C * cts + 2 * st + 4 * h * d * cts)
    if name == "global_bwd_carry":
        return chains * (5 * (h + d) * C * cts + 3 * st)
    if name == "local_carry":
        return local_carry_bytes(cfg)["alg_bytes"]
    return None


def local_carry_bytes(cfg):
    """Algorithmic HBM bytes of one local-memory walk (the state carry), averaged
    over the layer's local memories (one walk launch each).

    With the state resident on chip across the chunk loop the walk must read the
    chunk's keys and values (compute type) and its three gates (fp32), and write
    the chunk-entry state the backward needs (W1, W2, S1, S2 and the d x d Q-K
    sum, compute type): that is ``alg_bytes``.  ``spilled_state_bytes`` is what a
    walk that kept the fp32 state in memory would move on top (read and write
    4 h d fp32 per chunk)."""
    d, h = cfg.d, cfg.hid
    cts = 2 if cfg.dtype == 1 else 4
    alg = spill = 0
    for (C, S) in cfg.locals_:
        units = cfg.B * cfg.H * (cfg.L // S)
        nch = S // C
        per_chunk = 2 * C * d * cts + 3 * C * 4 + (4 * h * d + d * d) * cts
        alg += units * nch * per_chunk
        spill += units * nch * 2 * 4 * h * d * 4
    n = max(1, len(cfg.locals_))
    return {"alg_bytes": alg // n, "spilled_state_bytes": spill // n}


# labels timed inside another launch (reported separately, never the dominant launch)
SECTIONS = ("global_carry", "global_bwd_carry", "local_carry", "local_bwd_walk")


def launch_flops(cfg, name):
    """Algorithmic FLOPs one launch of `name` processes (None if not a GEMM kernel)."""
    tok = cfg.B * cfg.H * cfg.L
    C = cfg.locals_[0][0] if cfg.locals_ else 0
    if name == "local_fwd":
        return local_fwd_flops(cfg.d, cfg.hid, C, cfg.qk_proj) * tok
    if name == "local_bwd":
        return local_bwd_flops(cfg.d, cfg.hid, C, cfg.qk_proj) * tok
    per_chunk = cfg.B * cfg.H * cfg.C_G
    G = cfg.L // cfg.C_G
    dh = cfg.d * cfg.hid
    if name == "global_fwd_chunk":   # mean over the step's launches (the last chunk: its
        return (18 * dh * (G - 1) + 4 * dh) * per_chunk / G   # retrieval only)
    if name == "global_bwd_chunk":
        return global_bwd_flops(cfg.d, cfg.hid) * per_chunk
    return None


# ----------------------------------------------------------------------------
# measured HBM traffic of a launch (rocprofv3 FETCH_SIZE / WRITE_SIZE, calibrated
# against a plain copy; committed under profiles/), valid while the sources of
# the launch's kernels still hash to the recorded value
# ----------------------------------------------------------------------------
TRAFFIC_FILE = {2: "hbm_traffic_pretrain_B4H8L8192.txt"}
_COMMON = ["tnt_device.h", "tnt_kernels.h"]
LAUNCH_SOURCES = {
    "local_bwd": ["tnt_local_bwd_split.hip", "tnt_local_bwd_split.h", "tnt_local_bwd_walk.hip",
                  "tnt_local_bwd_helpers.h", "tnt_local_bwd_layout.h", "tnt_regtile.h",
                  "tnt_local_common.h", "tnt_local_record.h"] + _COMMON,
    "local_fwd": ["tnt_local_fwd_fast.hip", "tnt_local_walk.hip", "tnt_local_ret.hip", "tnt_regtile.h",
                  "tnt_local_common.h",
                  "tnt_local_record.h"] + _COMMON,
    "local_carry": ["tnt_local_walk.hip", "tnt_regtile.h", "tnt_local_common.h",
                    "tnt_local_record.h"] + _COMMON,
    "global_bwd_chunk": ["tnt_global_bwd.hip", "tnt_global_blk.hip"] + _COMMON,
    "global_fwd_chunk": ["tnt_global_fwd.hip", "tnt_global_blk.hip"] + _COMMON,
    "global_scan": ["tnt_global_fwd.hip"] + _COMMON,
    "global_carry": ["tnt_global_fwd.hip", "tnt_global_blk.hip"] + _COMMON,
    "global_bwd_carry": ["tnt_global_bwd.hip", "tnt_global_blk.hip"] + _COMMON,
}
MFMA_FILE = {2: "mfma_ops_pretrain_B4H8L8192.txt"}


def all_sources_hash():
    import hashlib
    h = hashlib.sha256()
    d = os.path.join(ROOT, "paper_2511_07343_amd", "csrc")
    for fn in sorted(os.listdir(d)):
        with open(os.path.join(d, fn), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_mfma(workload):
    """MFMA FLOPs per step counted by rocprofv3 (committed summary), or None
    once any kernel source changed since the count was taken."""
    fn = MFMA_FILE.get(workload)
    path = os.path.join(ROOT, "profiles", fn) if fn else None
    if not path or not os.path.exists(path):
        return None
    with open(path) as f:
        for line in f:
            t = line.split()
            if len(t) >= 6 and t[0] == "step" and t[1] == "sha256":
                return float(t[5]) if t[2] == all_sources_hash() else None
    return None


def sources_hash(label):
    import hashlib
    h = hashlib.sha256()
    for fn in LAUNCH_SOURCES[label]:
        with open(os.path.join(ROOT, "paper_2511_07343_amd", "csrc", fn), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic(workload, label):
    """HBM bytes per launch of `label` from the committed counter summary, or None."""
    fn = TRAFFIC_FILE.get(workload)
    if fn is None or label not in LAUNCH_SOURCES:
        return None
    path = os.path.join(ROOT, "profiles", fn)
    if not os.path.exists(path):
        return None
    with open(path) as f:
        for line in f:
            t = line.split()
            if len(t) >= 10 and t[0] == "launch" and t[1] == label:
                return float(t[9]) if t[3] == sources_hash(label) else None
    return None


# ----------------------------------------------------------------------------
def cpu_baseline(cfg, inp, budget_tokens):
    """fp64 oracle, fwd + bwd, on one (batch 0, head 0) chain restricted to its
    first `budget_tokens` tokens (the whole 8192-token chain, four local shards
    and four global chunks, at the default workload)."""
    import torch
    import oracle as O

    n = len(os.sched_getaffinity(0))
    torch.set_num_threads(n)
    L = budget_tokens
    sub = cfg.replace(L=L, B=1, H=1)
    g = O.gather_pairs(inp, [(0, 0)])
    cut = lambda t, ax: t.narrow(ax, 0, L).contiguous()
    args = [cut(g["q"], 1), cut(g["k"], 1), cut(g["v"], 1), cut(g["lr"], 2), cut(g["mom"], 2),
            cut(g["decay"], 2), g["W1"], g["W2"]]
    t0 = time.perf_counter()
    ref = O.layer_backward(*args, cut(g["dO"], 1), sub)
    dt = time.perf_counter() - t0
    return {"value": L / dt, "unit": "tokens/s", "cores": torch.get_num_threads(),
            "kind": "oracle",
            "sample": f"fwd+bwd of one (batch 0, head 0) chain, first {L} tokens "
                      f"(fp64 torch CPU autograd, {dt:.1f} s)"}, ref


def sample_parity(cfg, ref, o, g, L):
    """Per-tensor max |gpu - oracle| / max |oracle| of the timed run's last step on
    the oracle sample's chain (batch 0, head 0).  The outputs of a causal layer
    on the first L tokens do not depend on later tokens, so o is compared on any
    sample; the gradients only when the sample is the whole chain."""
    import numpy as np
    from paper_2511_07343_amd.inputs import max_rel_err
    got = {"o": o[0, 0, :L]}
    if L == cfg.L:
        for n in ("dq", "dk", "dv"):
            got[n] = g[n][0, 0]
        for n in ("dlr", "dmom", "ddecay"):
            got[n] = g[n][:, 0, 0]
    out = {}
    for n, t in got.items():
        want = ref[n].numpy()
        want = want[0] if n in ("o", "dq", "dk", "dv") else want[:, 0]
        mine = t.float().cpu().numpy()
        if n in ("dlr", "dmom", "ddecay"):   # each memory against its own scale
            out[n] = max(max_rel_err(mine[m], want[m]) for m in range(cfg.M))
        else:
            out[n] = max_rel_err(mine, want)
    return {"max_rel_err": out, "bound": 2e-2 if cfg.dtype == 1 else 1e-4,
            "pass": all(np.isfinite(v) and v <= (2e-2 if cfg.dtype == 1 else 1e-4)
                        for v in out.values()),
            "sample": f"chain (batch 0, head 0), tokens 0..{L - 1}, against the fp64 oracle"}


def decode_bench(args, cfg, x, dev):
    """Step-wise forward: `args.steps` calls of tnt_mem_step with `args.decode`
    tokens per chain each, continuing one carried state; one JSON line."""
    import torch
    from paper_2511_07343_amd import tnt

    T = args.decode
    M = cfg.has_global + len(cfg.locals_)
    state = torch.empty(tnt.tnt_mem_state_size(cfg), dtype=torch.uint8, device=dev)
    if tnt.tnt_mem_state_init(cfg, x["W1"], x["W2"], state):
        raise RuntimeError("tnt_mem_state_init failed")
    n_calls = args.warmup + args.steps
    if n_calls * T > cfg.L:
        raise SystemExit(f"--decode {T} x {n_calls} calls exceeds the workload's {cfg.L} tokens")
    cp = lambda t: t.clone(memory_format=torch.contiguous_format)
    pieces = []
    for c in range(n_calls):
        sl = slice(c * T, (c + 1) * T)
        pieces.append([cp(x[n][:, :, sl]) for n in ("q", "k", "v")] +
                      [cp(x[n][..., sl]) for n in ("lr", "mom", "decay")])
    o = torch.empty_like(pieces[0][0])
    stream = torch.cuda.current_stream(dev)

    def call(c):
        q, k, v, lr, mom, dec = pieces[c]
        st = tnt.tnt_mem_step(cfg, c * T, T, q, k, v, lr, mom, dec, x["W1"], x["W2"], state, o,
                              stream=stream)
        if st:
            raise tnt.TntError(st, "tnt_mem_step")

    for c in range(args.warmup):
        call(c)
    torch.cuda.synchronize()
    tnt.tnt_timing_read()
    tnt.tnt_timing_enable(True)
    t0 = time.perf_counter()
    for c in range(args.warmup, n_calls):
        call(c)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    tnt.tnt_timing_enable(False)
    kt = tnt.tnt_timing_read()
    ms_call = 1e3 * (t1 - t0) / args.steps
    ev_ms = kt["step"][0] / kt["step"][1]
    # per call and memory: read W^1, W^2, W1, W2, S1, S2, write W1, W2, S1, S2 (fp32); the
    # tokens of a call between two chunk starts can share them
    alg = M * cfg.B * cfg.H * 10 * cfg.hid * cfg.d * 4
    res = {
        "metric": f"step-wise forward tokens/s ({T} token(s) per chain per call)",
        "value": cfg.B * T * args.steps / (t1 - t0), "unit": "tokens/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_call,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f32 state, " + ("bf16" if cfg.dtype == inputs_bf16() else "f32") + " I/O",
        "data": "synthetic (seeded Gaussian, unit q/k)",
        "config": {"workload": cfg.name, "batch": cfg.B, "heads": cfg.H, "tokens_per_call": T},
        "roofline": {"bound": "hbm", "kernel": "step", "achieved": alg / (ev_ms * 1e-3) / 1e9,
                     "peak": PEAK_HBM / 1e9, "unit": "GB/s",
                     "frac": alg / (ev_ms * 1e-3) / PEAK_HBM, "traffic": None,
                     "avg_launch_ms": ev_ms, "alg_bytes_per_launch": alg},
    }
    print(json.dumps(res), flush=True)


def inputs_bf16():
    from paper_2511_07343_amd import inputs
    return inputs.BF16


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", type=int, default=2)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-tokens", type=int, default=0,
                    help="tokens of the CPU-oracle sample (default: one chain, at most "
                         "four local shards)")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="BYTES",
                    help="run one plain device copy of BYTES before the warmup (the "
                         "reference dispatch that scales HBM traffic counters)")
    ap.add_argument("--seq", type=int, default=0,
                    help="override the workload's sequence length (global chunk and local "
                         "shard are capped at it); the counter summaries then do not apply")
    ap.add_argument("--batch", type=int, default=0, help="override the workload's batch")
    ap.add_argument("--local-chunk", type=int, default=0, metavar="C",
                    help="override every local memory's chunk C_L (the small chunks of the "
                         "second training stage, C_L in {1, 2, 4}); the counter summaries then "
                         "do not apply")
    ap.add_argument("--decode", type=int, default=0, metavar="T",
                    help="time the step-wise forward (tnt_mem_step) with T tokens per chain "
                         "per call instead of the fwd+bwd step")
    ap.add_argument("--mfma-probe", type=int, default=0, metavar="N",
                    help="run one N x N x N bf16 matmul before the warmup (the reference "
                         "dispatch that scales MFMA operation counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only; --gpus {args.gpus} is not supported "
              "(the layer's multi-GPU split is a design note, not built)", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2511_07343_amd import inputs, tnt

    cfg = inputs.WORKLOADS[args.workload]
    seed = args.workload
    prof_key = args.workload  # committed counter summaries describe the unmodified workloads
    if args.seq or args.batch or args.local_chunk:
        import dataclasses
        L = args.seq or cfg.L
        B = args.batch or cfg.B
        loc = tuple((args.local_chunk or c, min(s_, L)) for c, s_ in cfg.locals_)
        cfg = dataclasses.replace(
            cfg, B=B, L=L, C_G=min(cfg.C_G, L), locals_=loc,
            name=f"{cfg.name.split(' B')[0]} B{B} H{cfg.H} L{L} d{cfg.d} h{cfg.hid} "
                 f"CG{min(cfg.C_G, L)} " + " ".join(f"CL{c} SL{s_}" for c, s_ in loc))
        prof_key = None
    inp = inputs.make_inputs(cfg, seed)
    dev = torch.device("cuda:0")
    x = tnt.device_inputs(inp, cfg, device=dev)
    if args.decode:
        return decode_bench(args, cfg, x, dev)
    u8 = lambda n: torch.empty(max(n, 16), dtype=torch.uint8, device=dev)
    o = torch.empty_like(x["q"])
    saved = u8(tnt.tnt_mem_saved_size(cfg))
    ws_f = u8(tnt.tnt_mem_workspace_size(cfg, tnt.TNT_WS_FWD))
    ws_b = u8(tnt.tnt_mem_workspace_size(cfg, tnt.TNT_WS_BWD))
    g = {k: torch.empty_like(x[s]) for k, s in
         (("dq", "q"), ("dk", "k"), ("dv", "v"), ("dlr", "lr"), ("dmom", "mom"),
          ("ddecay", "decay"), ("dW1", "W1"), ("dW2", "W2"))}
    stream = torch.cuda.current_stream(dev)
    if args.copy_probe:
        src = torch.ones(args.copy_probe, dtype=torch.uint8, device=dev)
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if args.mfma_probe:
        n = args.mfma_probe
        a_ = torch.ones(n, n, dtype=torch.bfloat16, device=dev)
        b_ = torch.ones(n, n, dtype=torch.bfloat16, device=dev)
        torch.matmul(a_, b_)
        torch.cuda.synchronize()
        del a_, b_

    def step():
        s1 = tnt.tnt_mem_fwd(cfg, x["q"], x["k"], x["v"], x["lr"], x["mom"], x["decay"], x["W1"],
                             x["W2"], o, None, saved, ws_f, stream=stream)
        s2 = tnt.tnt_mem_bwd(cfg, x["q"], x["k"], x["v"], x["lr"], x["mom"], x["decay"],
                             x["W1"], x["W2"], x["dO"], saved, g["dq"], g["dk"], g["dv"],
                             g["dlr"], g["dmom"], g["ddecay"], g["dW1"], g["dW2"], ws_b,
                             stream=stream)
        if s1 or s2:
            raise tnt.TntError(s1 or s2, "step")

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    # The timed region: K steps with nothing but the layer's own launches; per-step
    # events on the caller's stream (the helper streams fork from and join back
    # into it inside every call, so they bracket the whole step).
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    t0 = time.perf_counter()
    evs[0].record(stream)
    for i in range(args.steps):
        step()
        evs[i + 1].record(stream)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    per_step = sorted(evs[i].elapsed_time(evs[i + 1]) for i in range(args.steps))
    median_ms = per_step[len(per_step) // 2] if len(per_step) % 2 else \
        0.5 * (per_step[len(per_step) // 2 - 1] + per_step[len(per_step) // 2])
    # Per-launch times from a second run of K steps with an event pair around
    # every launch (on the stream it runs on).  The pairs cost about 0.13 ms a
    # step at workload 2, so they stay out of the timed region.
    tnt.tnt_timing_read()
    tnt.tnt_timing_enable(True)
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    tnt.tnt_timing_enable(False)
    kt = tnt.tnt_timing_read()
    assert torch.isfinite(o.float()).all() and torch.isfinite(g["dq"].float()).all()
    if "local_bwd_gate" in kt and "local_bwd" in kt:
        # the last local memory's gate pass, launched after the global chain, is part
        # of that memory's backward launch
        gt, _ = kt.pop("local_bwd_gate")
        kt["local_bwd"] = (kt["local_bwd"][0] + gt, kt["local_bwd"][1])

    elapsed = t1 - t0
    ms_step = 1e3 * elapsed / args.steps
    tokens = cfg.B * cfg.L
    value = tokens * args.steps / elapsed
    flops = step_flops(cfg)
    bf = cfg.dtype == inputs.BF16
    peak = PEAK_BF16 if bf else PEAK_FP32

    # dominant kernel by total event time in the timed region
    dom = max(((k, v) for k, v in kt.items() if k not in SECTIONS), key=lambda kv: kv[1][0])
    name, (tot_ms, n) = dom
    fl = launch_flops(cfg, name)
    avg_ms = tot_ms / n
    roof = {"bound": "mfma", "kernel": name, "achieved": None, "peak": peak / 1e12,
            "unit": "TFLOP/s", "frac": None, "traffic": None, "avg_launch_ms": avg_ms,
            "launches": n}
    if fl is not None:
        ach = fl / (avg_ms * 1e-3) / 1e12
        roof.update(achieved=ach, frac=ach * 1e12 / peak, flops_per_launch=fl)
    roof["traffic"] = measured_traffic(prof_key, name)
    # HBM-bound steps: the gate scan and the global state carry (forward, backward)
    hbm = {}
    for lab in ("global_scan",) + SECTIONS:
        if lab not in kt or hbm_bytes(cfg, lab) is None or lab == "local_carry":
            continue
        t_ms, n_l = kt[lab]
        avg = t_ms / n_l
        ab = hbm_bytes(cfg, lab)
        tb = measured_traffic(prof_key, lab)
        hbm[lab] = {"avg_launch_ms": avg, "launches": n_l, "alg_bytes": ab,
                    "alg_GBps": ab / (avg * 1e-3) / 1e9,
                    "alg_frac": ab / (avg * 1e-3) / PEAK_HBM,
                    "counter_bytes": tb,
                    "counter_GBps": None if tb is None else tb / (avg * 1e-3) / 1e9,
                    "peak_GBps": PEAK_HBM / 1e9}
    carry = None
    if "local_carry" in kt and cfg.locals_:
        t_ms, n_l = kt["local_carry"]
        avg = t_ms / n_l
        cb = local_carry_bytes(cfg)
        tb = measured_traffic(prof_key, "local_carry")
        carry = {"avg_launch_ms": avg, "launches": n_l, "alg_bytes": cb["alg_bytes"],
                 "alg_GBps": cb["alg_bytes"] / (avg * 1e-3) / 1e9,
                 "alg_frac": cb["alg_bytes"] / (avg * 1e-3) / PEAK_HBM,
                 "state": "resident (registers) across the chunk loop",
                 "spilled_state_bytes_avoided": cb["spilled_state_bytes"],
                 "counter_bytes": tb,
                 "counter_GBps": None if tb is None else tb / (avg * 1e-3) / 1e9,
                 "peak_GBps": PEAK_HBM / 1e9}
    mf = measured_mfma(prof_key)
    mfma = None
    if mf is not None:
        mfma = {"flops_per_step": mf, "tflops": mf / (ms_step * 1e-3) / 1e12,
                "frac": mf / (ms_step * 1e-3) / peak, "source": "rocprofv3 PMC "
                "SQ_INSTS_VALU_MFMA_MOPS_BF16 + _F32, scaled by a known bf16 GEMM"}
    props = torch.cuda.get_device_properties(dev)
    clk = getattr(props, "clock_rate", None)
    device = {"name": props.name, "compute_units": props.multi_processor_count,
              "clock_mhz": (clk / 1e3) if clk else None,
              "peak_used_tflops": peak / 1e12,
              "peak_note": "published MI355X dense peak (bf16 MFMA 2.5 PFLOP/s, fp32 157.3 TFLOP/s)"}

    res = {
        "metric": METRIC, "value": value, "unit": "tokens/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_step,
        "median_ms_per_step": median_ms, "min_ms_per_step": per_step[0],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16" if bf else "f32", "data": "synthetic (seeded Gaussian, unit q/k)",
        "config": {"workload": cfg.name, "global_batch": cfg.B, "seq_len": cfg.L,
                   "heads": cfg.H, "head_dim": cfg.d, "hidden": cfg.hid, "C_G": cfg.C_G,
                   "locals": [list(t) for t in cfg.locals_], "parallelism": "single GPU"},
        "algorithmic_tflops": flops / elapsed * args.steps / 1e12,
        "algorithmic_frac_of_peak": flops / elapsed * args.steps / peak,
        "roofline": roof,
        "paper_context": PAPER_CONTEXT,
        "mfma_counted": mfma,
        "hbm_kernels": hbm,
        "local_state_carry": carry,
        "sections_ms_per_step": {k: v[0] / args.steps for k, v in sorted(kt.items())
                                 if k in SECTIONS},
        "device": device,
        "kernels_ms_per_step": {k: v[0] / args.steps for k, v in sorted(kt.items())
                                if k not in SECTIONS},
    }
    if not args.no_cpu_baseline:
        unit = cfg.locals_[0][1] if cfg.locals_ else cfg.C_G
        ctoks = args.cpu_tokens or min(cfg.L, 4 * unit)
        res["cpu_baseline"], ref = cpu_baseline(cfg, inp, ctoks)
        res["parity"] = sample_parity(cfg, ref, o, g, ctoks)
    print(json.dumps(res), flush=True)


if __name__ == "__main__":
    main()
