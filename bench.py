#!/usr/bin/env python3
"""Benchmark of the gated group rollout on one MI355X.

A "step" is one turn of the episode: an observation chunk is prefilled for every live sequence,
act_len tokens are decoded greedily, and at the gate turn the gate runs and retired groups are
compacted out.  The shared prompt prefill that opens the episode is inside the timed region.
Inputs are seeded and synthetic (random-init Qwen2.5-7B-shaped decoder, uniform token ids); they
stand in for the paper's ALFWorld / Qwen2.5-7B-Instruct rollouts, which are not reproduced here.

Prints ONE JSON line: decoded tokens/s for the whole job, the HBM roofline of the dominant kernel
(the decode-time gate|up projection with SwiGLU epilogue, timed with HIP events on the stream it
runs on), the per-decode-step HBM fraction, gate throughput, and the CPU checker timed on a
bounded sample of the same workload.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # published HBM3E peak of the MI355X
MFMA_PEAK_TFLOPS = 2500.0      # published dense bf16 matrix-core peak


def measured_peaks(sr, torch):
    """What the chip this run is on achieves with nothing in the way: a streaming read of 4 GiB (with the
    non-temporal loads the weight-streaming kernels use, and with default loads), a plain copy, and a
    register-resident bf16 matrix-core loop.  Quoted next to the published peaks."""
    buf = torch.zeros(1 << 30, dtype=torch.int32, device="cuda")        # 4 GiB: far beyond every cache
    dst = torch.empty(1 << 28, dtype=torch.int32, device="cuda")
    out = {"hbm_read_nt_GBs": sr.sr_probe_hbm(buf, dst, 0),
           "hbm_read_GBs": sr.sr_probe_hbm(buf, dst, 1)}
    out["hbm_copy_GBs"] = sr.sr_probe_hbm(buf[:1 << 28], dst, 2)
    out["mfma_bf16_TFLOPs"] = sr.sr_probe_mfma_bf16(dst)
    del buf, dst
    torch.cuda.empty_cache()
    return out


def weight_bytes_per_step(s) -> int:
    per_layer = s.hidden * (s.q_dim + 2 * s.kv_dim) + s.q_dim * s.hidden + 3 * s.hidden * s.ffn
    return 2 * (s.n_layers * per_layer + s.vocab * s.hidden)


def kv_bytes_per_token(s) -> int:
    return 2 * s.n_kv_heads * s.head_dim * 2 * s.n_layers


def run_episode(sr, torch, synth, shape, cfg, weights, turns, seed, profile_step):
    """One gated episode through the C boundary.  Returns timings and counters."""
    G = cfg.G
    max_len = cfg.prompt_len + cfg.turns * (cfg.obs_len + cfg.act_len)
    kv_tokens = cfg.n_groups * cfg.prompt_len + cfg.n_groups * G * (max_len - cfg.prompt_len + 64)
    pool = int(kv_tokens * kv_bytes_per_token(shape) * 1.05) + (64 << 20)
    ctx = sr.Context(shape, cfg.n_groups, G, cfg.threshold, page_tokens=64, max_seq_len=max_len,
                     max_turns=cfg.turns, action_mod=cfg.action_mod, kv_pool_bytes=pool)
    embed, lm, fn, layers = weights
    ctx.sr_load_weights(embed, lm, fn, layers)

    conv = synth.converging_groups(cfg, seed)
    prompts = torch.from_numpy(synth.prompts(cfg, shape.vocab, seed)).cuda()
    obs_all = [synth.observations(cfg, shape.vocab, seed, t, conv) for t in range(turns)]
    live_rows = np.arange(cfg.n_groups * G)

    torch.cuda.synchronize()
    ev = lambda: torch.cuda.Event(enable_timing=True)
    step_events, decode_meta, prefill_events = [], [], []
    t0 = time.perf_counter()
    ctx.sr_prefill_chunk(prompts, True)
    for turn in range(turns):
        obs = torch.from_numpy(obs_all[turn][live_rows]).cuda()
        p0, p1 = ev(), ev()
        p0.record()
        ctx.sr_prefill_chunk(obs, False)
        p1.record()
        prefill_events.append((p0, p1, len(live_rows) * cfg.obs_len))
        for a in range(cfg.act_len):
            prof = profile_step is not None and a == profile_step
            if prof:
                ctx.sr_profile(True)
            e0, e1 = ev(), ev()
            e0.record()
            ctx.sr_decode_step()
            e1.record()
            if prof:
                ctx.sr_profile(False)
            st_len = cfg.prompt_len + turn * (cfg.obs_len + cfg.act_len) + cfg.obs_len + a + 1
            step_events.append((e0, e1))
            decode_meta.append((len(live_rows), st_len, prof))
        if (turn + 1) in cfg.gate_turns:
            ctx.sr_gate(turn + 1)
            ctx.sr_retire_and_compact()
            live_rows = ctx.sr_get_live_map()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    kernel_times = ctx.sr_profile_read() if profile_step is not None else {}
    stats = ctx.sr_stats()
    step_ms = [a.elapsed_time(b) for a, b in step_events]
    ctx.close()
    prefill = [(a.elapsed_time(b), rows) for a, b, rows in prefill_events]
    return {"wall_s": wall, "stats": stats, "step_ms": step_ms, "decode_meta": decode_meta, "prefill": prefill,
            "kernel_times": kernel_times, "shared_tokens": (cfg.prompt_len // 64) * 64}


def score_pass(sr, torch, synth, shape, cfg, weights, turns, seed):
    """Teacher-forced log-likelihood pass (Appendix C.2) over trajectories of the benchmark's shape: prompt and
    observations go through sr_prefill_chunk, the action tokens of every turn through sr_score_chunk."""
    G = cfg.G
    max_len = cfg.prompt_len + cfg.turns * (cfg.obs_len + cfg.act_len)
    kv_tokens = cfg.n_groups * cfg.prompt_len + cfg.n_groups * G * (max_len - cfg.prompt_len + 64)
    pool = int(kv_tokens * kv_bytes_per_token(shape) * 1.05) + (64 << 20)
    ctx = sr.Context(shape, cfg.n_groups, G, cfg.threshold, page_tokens=64, max_seq_len=max_len,
                     max_turns=cfg.turns, action_mod=cfg.action_mod, kv_pool_bytes=pool)
    embed, lm, fn, layers = weights
    ctx.sr_load_weights(embed, lm, fn, layers)
    conv = synth.converging_groups(cfg, seed)
    prompts = torch.from_numpy(synth.prompts(cfg, shape.vocab, seed)).cuda()
    n_seq = cfg.n_groups * G
    gen = torch.Generator(device="cuda").manual_seed(seed)
    ctx.sr_prefill_chunk(prompts, True)
    obs_all = [torch.from_numpy(synth.observations(cfg, shape.vocab, seed, t, conv)).cuda() for t in range(turns)]
    acts_all = [torch.randint(0, shape.vocab, (n_seq, cfg.act_len), dtype=torch.int32, device="cuda", generator=gen)
                for _ in range(turns)]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    score_ms = 0.0
    evs = []
    for t in range(turns):
        ctx.sr_prefill_chunk(obs_all[t], False)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        ctx.sr_score_chunk(acts_all[t])
        e1.record()
        evs.append((e0, e1))
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    score_ms = sum(a.elapsed_time(b) for a, b in evs)
    ctx.close()
    n_act = n_seq * cfg.act_len * turns
    flops_lm = 2.0 * shape.hidden * shape.vocab * n_act
    flops_body = 2.0 * (weight_bytes_per_step(shape) / 2 - shape.hidden * shape.vocab) * n_act
    return {"action_tokens": n_act, "action_tokens_per_s": n_act / wall, "wall_s": wall,
            "score_calls_ms": score_ms, "score_calls_TFLOPs": (flops_lm + flops_body) / (score_ms * 1e-3) / 1e12,
            "note": "wall includes the observation prefills; score_calls_* cover sr_score_chunk only "
                    "(transformer body + LM head on every action row + log-softmax gather)"}


def sampling_steps(sr, torch, synth, shape, cfg, weights, seed, temperature=0.7, steps=8):
    """Token selection at the paper's rollout temperature (Section 3.1): a few decode steps of the benchmark's batch
    with Gumbel-max sampling, timed per kernel class, next to the same steps decoded greedily."""
    G = cfg.G
    max_len = cfg.prompt_len + cfg.obs_len + steps + 64
    kv_tokens = cfg.n_groups * cfg.prompt_len + cfg.n_groups * G * (max_len - cfg.prompt_len + 64)
    pool = int(kv_tokens * kv_bytes_per_token(shape) * 1.05) + (64 << 20)
    out = {}
    for name, temp in (("greedy", 0.0), ("sampled", temperature)):
        ctx = sr.Context(shape, cfg.n_groups, G, cfg.threshold, page_tokens=64, max_seq_len=max_len, max_turns=4,
                         action_mod=cfg.action_mod, kv_pool_bytes=pool, temperature=temp, sample_seed=seed)
        embed, lm, fn, layers = weights
        ctx.sr_load_weights(embed, lm, fn, layers)
        conv = synth.converging_groups(cfg, seed)
        ctx.sr_prefill_chunk(torch.from_numpy(synth.prompts(cfg, shape.vocab, seed)).cuda(), True)
        ctx.sr_prefill_chunk(torch.from_numpy(synth.observations(cfg, shape.vocab, seed, 0, conv)).cuda(), False)
        ctx.sr_decode_step()
        ctx.sr_profile(True)
        for _ in range(steps):
            ctx.sr_decode_step()
        ctx.sr_profile(False)
        kt = ctx.sr_profile_read()
        ctx.close()
        out[name + "_select_ms_per_step"] = kt["argmax"][1] / steps
        out[name + "_step_ms"] = sum(v[1] for v in kt.values()) / steps
    out["temperature"] = temperature
    out["note"] = "select = one kernel over [rows][vocab] fp32 logits: argmax, or argmax of logit/T + Gumbel noise"
    return out


def gate_throughput(sr, torch, synth, iters=20):
    acts, _ = synth.gate_actions(65536, 8, 30, 64, seed=0)
    a = torch.from_numpy(acts).cuda()
    sums = torch.empty((3, 65536), dtype=torch.int32, device="cuda")
    ret = torch.empty((3, 65536), dtype=torch.uint8, device="cuda")
    for _ in range(3):
        sr.sr_gate_batch(a, [5, 10, 15], 0.3, sums, ret)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(iters):
        sr.sr_gate_batch(a, [5, 10, 15], 0.3, sums, ret)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / iters
    # the same by the other decomposition (one workgroup per group, anti-diagonals in LDS), for comparison
    for _ in range(3):
        sr.sr_gate_batch_antidiag(a, [5, 10, 15], 0.3, sums, ret)
    e0.record()
    for _ in range(iters):
        sr.sr_gate_batch_antidiag(a, [5, 10, 15], 0.3, sums, ret)
    e1.record()
    torch.cuda.synchronize()
    ms_ad = e0.elapsed_time(e1) / iters
    return 65536 / (ms * 1e-3), ms, acts, ms_ad


def signals_throughput(sr, torch, acts, iters=20):
    """Appendix-B signals and the two-clause gate on the same 65536 groups, with early finishers."""
    rng = np.random.default_rng(1)
    n_groups, G, stride = acts.shape
    obs = rng.integers(0, 3, size=acts.shape).astype(np.int32)
    end = np.where(rng.random((n_groups, G)) < 0.35, rng.integers(1, stride + 1, size=(n_groups, G)),
                   10 ** 6).astype(np.int32)
    a, o, e = torch.from_numpy(acts).cuda(), torch.from_numpy(obs).cuda(), torch.from_numpy(end).cuda()
    out = torch.zeros((3, n_groups, sr.SIGNALS_BYTES), dtype=torch.uint8, device="cuda")
    lens = [5, 10, 15]
    for _ in range(3):
        sr.sr_signals_batch(a, lens, 0.12, 0.9, out, obs=o, end_step=e)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(iters):
        sr.sr_signals_batch(a, lens, 0.12, 0.9, out, obs=o, end_step=e)
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / iters
    return n_groups / (ms * 1e-3), ms


def cpu_baseline(synth, shape, cfg, acts, turns=2):
    """The CPU checker, as it stands, on a bounded sample of the same workload:
      - the gate workload in full (65536 groups, prefixes 5/10/15) and the signals on the same groups;
      - the tiny configuration's gated episode in full (4 groups x 8, 6 turns);
      - one sequence of the benchmark's model shape (weights from the same seeded generator, on the host) through
        `turns` turns: its share of the group's prompt, then per turn the observation chunk and the action tokens
        one by one.  A 1024-token prompt alone would cost the checker about 70 s (1024 tokens x 14.1 GFLOP at the
        measured rate), beyond the 10-30 s this leg may take, so the slice's context stays near 200 tokens; what
        that leaves out is attention over a longer context, 0.4 MFLOP per context token against 14.1 GFLOP of
        projections per decoded token (3 % at 1024 tokens, 8 % at 2944)."""
    import oracle
    t0 = time.perf_counter()
    w = synth.make_weights(shape, seed=0)
    gen_s = time.perf_counter() - t0
    model = oracle.Model(w)
    # a member's share of the shared prompt, per turn of the whole episode
    prompt_share = max(1, round(cfg.prompt_len * turns / (cfg.G * cfg.turns)))
    n_fwd = prompt_share + turns * (cfg.obs_len + cfg.act_len)
    seq = model.new_seq(n_fwd + 2)
    toks = synth.uniform_ids(n_fwd + 1, 0, 777, shape.vocab)
    seq.forward(toks[:1])                                   # page the weights in
    pos = 1
    t0 = time.perf_counter()
    seq.forward(toks[pos:pos + prompt_share])
    pos += prompt_share
    dec_s = 0.0
    for _ in range(turns):
        seq.forward(toks[pos:pos + cfg.obs_len])
        pos += cfg.obs_len
        t1 = time.perf_counter()
        for t in toks[pos:pos + cfg.act_len]:
            seq.forward([t])
        dec_s += time.perf_counter() - t1
        pos += cfg.act_len
    dt = time.perf_counter() - t0
    decoded = turns * cfg.act_len
    tok_s = decoded / dt
    del model, seq, w

    n_groups = acts.shape[0]
    t0 = time.perf_counter()
    oracle.gate_batch(acts, [5, 10, 15], 0.3)
    gate_dt = time.perf_counter() - t0
    rng = np.random.default_rng(1)
    end = np.where(rng.random((n_groups, acts.shape[1])) < 0.35,
                   rng.integers(1, acts.shape[2] + 1, size=(n_groups, acts.shape[1])), 10 ** 6).astype(np.int32)
    t0 = time.perf_counter()
    oracle.signals_batch(acts, [5, 10, 15], 0.12, 0.9, obs=acts, end_step=end)
    sig_dt = time.perf_counter() - t0

    tcfg, tshape = synth.TINY_EPISODE, synth.TINY
    tw = synth.make_weights(tshape, seed=0)
    tconv = synth.converging_groups(tcfg, 0)
    t0 = time.perf_counter()
    trec = oracle.run_episode(oracle.Model(tw), synth.prompts(tcfg, tshape.vocab, 0),
                              lambda t: synth.observations(tcfg, tshape.vocab, 0, t, tconv), tcfg.G, tcfg.turns,
                              tcfg.act_len, tcfg.action_mod, tcfg.gate_turns, tcfg.threshold)
    tiny_dt = time.perf_counter() - t0

    cores = len(os.sched_getaffinity(0))
    threads = int(os.environ.get("OMP_NUM_THREADS", cores))
    return {"value": tok_s, "unit": "decoded tokens/s", "cores": min(threads, cores) if threads else cores,
            "kind": "oracle",
            "sample": f"one sequence of the benchmark's model shape in fp64: {prompt_share} prompt tokens (a member's "
                      f"share of the group prompt for {turns} of {cfg.turns} turns), then {turns} turns of {cfg.obs_len} "
                      f"observation + {cfg.act_len} decoded tokens; value = decoded tokens / whole-sample time "
                      f"({dt:.1f} s); a 1024-token context is not reached: the prompt alone would take about "
                      f"{1024 * dt / n_fwd:.0f} s; gate and signals: all {n_groups} groups of the gate workload; tiny "
                      f"configuration: its whole gated episode",
            "decode_only_tokens_per_s": decoded / dec_s,
            "gate_groups_per_s": n_groups / gate_dt, "gate_s": gate_dt,
            "signals_groups_per_s": n_groups / sig_dt, "signals_s": sig_dt,
            "tiny_episode_decoded_tokens_per_s": trec["decoded_tokens"] / tiny_dt, "tiny_episode_s": tiny_dt,
            "weight_generation_s": gen_s}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--workload", default="7b-g8-16groups",
                    choices=["7b-g8-16groups", "tiny", "7b-g8-64groups", "7b-g16-32groups"],
                    help="default: the configuration the metric is quoted on; the two larger ones (512 sequences, "
                         "90 and 120 GB of KV) are optional extra runs")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-score-pass", action="store_true", help="skip the teacher-forced scoring pass (extra object)")
    ap.add_argument("--layers", type=int, default=0,
                    help="counter collection only: truncate the model to this many layers (not a valid headline run)")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run one plain 1 GiB device copy (reference for scaling HBM traffic counters)")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: the library runs on one GPU only (groups are independent: the path would shard by "
              "partitioning groups over GPUs with replicated weights and no collective). Run with --gpus 1.",
              file=sys.stderr)
        sys.exit(2)

    import torch
    import paper_2605_05802_amd as sr
    import synth
    if not torch.cuda.is_available():
        print("bench.py: no GPU visible; the HIP path has no CPU fallback", file=sys.stderr)
        sys.exit(3)
    sr.lib()

    if args.workload == "tiny":
        shape, cfg = synth.TINY, synth.TINY_EPISODE
    elif args.workload == "7b-g8-64groups":
        shape, cfg = synth.QWEN7B, synth.C4_EPISODE
    elif args.workload == "7b-g16-32groups":
        shape, cfg = synth.QWEN7B, synth.C5_EPISODE
    else:
        shape, cfg = synth.QWEN7B, synth.C3_EPISODE
    turns = min(args.steps, cfg.turns)
    if args.layers > 0:
        import dataclasses
        shape = dataclasses.replace(shape, n_layers=args.layers)
        cfg = dataclasses.replace(cfg, prompt_len=64)

    if args.calibrate_copy:
        src = torch.zeros(1 << 28, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)                      # reads 1 GiB, writes 1 GiB
        torch.cuda.synchronize()
        del src, dst
    print("bench: measuring the chip's ceilings", file=sys.stderr, flush=True)
    peaks = measured_peaks(sr, torch)
    print("bench: generating weights", file=sys.stderr, flush=True)
    weights = synth.make_weights_device(shape, seed=0)
    print("bench: running", file=sys.stderr, flush=True)
    if args.warmup > 0:
        run_episode(sr, torch, synth, shape, cfg, weights, min(args.warmup, cfg.turns), 0, None)
    res = run_episode(sr, torch, synth, shape, cfg, weights, turns, 0, profile_step=cfg.act_len // 2)
    score = (score_pass(sr, torch, synth, shape, cfg, weights, turns, 0)
             if args.layers == 0 and not args.no_score_pass and args.workload in ("7b-g8-16groups", "tiny") else None)
    sampling = (sampling_steps(sr, torch, synth, shape, cfg, weights, 0)
                if args.layers == 0 and args.workload in ("7b-g8-16groups", "tiny") else None)
    del weights
    torch.cuda.empty_cache()

    decoded = res["stats"]["decoded_tokens"]
    wall = res["wall_s"]
    # dominant kernel: decode-time gate|up projection (SwiGLU epilogue)
    launches, total_ms = res["kernel_times"]["gemm_gate_up"]
    avg_ms = total_ms / max(launches, 1)
    rows = [m for m in res["decode_meta"] if m[2]]
    mean_rows = float(np.mean([m[0] for m in rows])) if rows else 0.0
    gu_bytes = 2 * (2 * shape.ffn * shape.hidden) + mean_rows * shape.hidden * 2 + mean_rows * shape.ffn * 2
    achieved = gu_bytes / (avg_ms * 1e-3) / 1e9 if avg_ms > 0 else 0.0
    roofline = {"bound": "hbm", "kernel": "gemm_stream_kernel<EPI_SWIGLU, 5, MT32, 8> (decode gate|up projection)",
                "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS,
                "peak_measured": peaks["hbm_read_nt_GBs"], "frac_of_measured": achieved / peaks["hbm_read_nt_GBs"]}
    if mean_rows > 256:
        # more than 256 rows per step: the projection runs on a tiled kernel and is bound by the matrix cores
        tf = 2.0 * mean_rows * 2 * shape.ffn * shape.hidden / (avg_ms * 1e-3) / 1e12 if avg_ms > 0 else 0.0
        roofline = {"bound": "mfma", "kernel": "decode gate|up projection at more than 256 rows (tiled kernels)",
                    "achieved": tf, "peak": MFMA_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": tf / MFMA_PEAK_TFLOPS,
                    "peak_measured": peaks["mfma_bf16_TFLOPs"], "frac_of_measured": tf / peaks["mfma_bf16_TFLOPs"]}
    traffic = None
    tpath = os.path.join(ROOT, "profiles", "traffic.json")
    if os.path.exists(tpath):
        import hashlib
        t = json.load(open(tpath))
        src = open(os.path.join(ROOT, "paper_2605_05802_amd", "csrc", "gemm_stream.hip"), "rb").read()
        if t.get("kernel_source_sha1") == hashlib.sha1(src).hexdigest() and args.workload != "tiny":
            traffic = t.get("gate_up_decode_bytes_per_launch")

    # whole decode step against the HBM roofline (un-profiled steps only)
    wb, kvb = weight_bytes_per_step(shape), kv_bytes_per_token(shape)
    fr, gbs = [], []
    for (n_rows, st_len, prof), ms in zip(res["decode_meta"], res["step_ms"]):
        if prof:
            continue
        n_groups = n_rows // cfg.G
        kv_read = kvb * (n_groups * res["shared_tokens"] + n_rows * (st_len - res["shared_tokens"]))
        b = wb + kv_read + kvb * n_rows + 2 * n_rows * shape.vocab * 4
        gbs.append(b / (ms * 1e-3) / 1e9)
    step_ms = [ms for (m, ms) in zip(res["decode_meta"], res["step_ms"]) if not m[2]]

    # observation prefill against the matrix peak: projection flops only (attention not counted)
    layer_params = shape.hidden * (shape.n_q_heads + 2 * shape.n_kv_heads) * shape.head_dim \
        + shape.n_q_heads * shape.head_dim * shape.hidden + 3 * shape.hidden * shape.ffn
    pf_rate = [2.0 * layer_params * shape.n_layers * rows / (ms * 1e-3) / 1e12 for ms, rows in res["prefill"]]
    prefill_obj = {"ms_median": float(np.median([ms for ms, _ in res["prefill"]])),
                   "projection_TFLOPs_median": float(np.median(pf_rate)),
                   "frac_of_bf16_mfma_peak": float(np.median(pf_rate)) / MFMA_PEAK_TFLOPS,
                   "frac_of_measured_mfma_peak": float(np.median(pf_rate)) / peaks["mfma_bf16_TFLOPs"],
                   "rows_first_turn": res["prefill"][0][1]} if res["prefill"] else None

    gate_gps, gate_ms, acts, gate_ms_ad = gate_throughput(sr, torch, synth)
    sig_gps, sig_ms = signals_throughput(sr, torch, acts)
    out = {
        "metric": f"decoded tokens/s at Qwen2.5-7B shape, G={cfg.G} (whole gated episode: prompt prefill, per-turn "
                  "observation prefill, greedy decode, gate, compaction)",
        "value": decoded / wall, "unit": "tokens/s", "n_gpus": 1, "steps": turns, "warmup": args.warmup,
        "ms_per_step": 1e3 * wall / turns, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": cfg.name, "layers": shape.n_layers, "hidden": shape.hidden, "groups": cfg.n_groups,
                   "G": cfg.G, "prompt": cfg.prompt_len, "turns": turns, "obs": cfg.obs_len, "act": cfg.act_len,
                   "gate_turns": list(cfg.gate_turns), "threshold": cfg.threshold},
        "roofline": dict(roofline, traffic=traffic if mean_rows <= 128 else None,
                         traffic_stored=traffic is not None and mean_rows <= 128, avg_launch_ms=avg_ms,
                         launches_timed=launches, algorithmic_bytes_per_launch=gu_bytes,
                         note="the dominant kernel alone; the whole decode step against the same peak is "
                              "decode_step.hbm_frac_median; traffic is a stored counter reading "
                              "(profiles/traffic.json), valid while the kernel source is unchanged"),
        "peaks": {"hbm_GBs_published": HBM_PEAK_GBS, "mfma_bf16_TFLOPs_published": MFMA_PEAK_TFLOPS, **peaks},
        "decode_step": {"ms_median": float(np.median(step_ms)), "ms_min": float(np.min(step_ms)),
                        "hbm_GBs_median": float(np.median(gbs)), "hbm_frac_median": float(np.median(gbs)) / HBM_PEAK_GBS,
                        "hbm_frac_best": float(np.max(gbs)) / HBM_PEAK_GBS,
                        "hbm_frac_of_measured_median": float(np.median(gbs)) / peaks["hbm_read_nt_GBs"],
                        "decode_only_tokens_per_s": decoded / (sum(res["step_ms"]) * 1e-3)},
        "prefill_chunk": prefill_obj,
        "kernel_ms_per_profiled_step": {k: v[1] / max(len(rows), 1) for k, v in res["kernel_times"].items()},
        "gate": {"groups_per_s": gate_gps, "ms_per_launch": gate_ms, "workload": "65536 groups x G=8, prefixes 5/10/15",
                 "kernel": "a lane per two pairs, bit-parallel table rows, equality masks from LDS",
                 "antidiagonal_lds_variant_ms_per_launch": gate_ms_ad,
                 "antidiagonal_lds_variant_groups_per_s": 65536 / (gate_ms_ad * 1e-3)},
        "score_pass": score,
        "sampling": sampling,
        "signals": {"groups_per_s": sig_gps, "ms_per_launch": sig_ms,
                    "workload": "same groups, 35 % of members finished early: Appendix-B signals + two-clause gate"},
        "episode": {k: res["stats"][k] for k in ("decoded_tokens", "prefill_tokens", "groups_retired", "pages_freed",
                                                "n_live_groups")},
        "paper_context": "paper reports wall-clock only (vLLM on RTX 6000 Ada): ~95% of time in rollout, ~40% "
                         "zero-variance groups, 10.7% end-to-end saving; not comparable numbers",
    }
    if not args.no_cpu_baseline:
        cshape = shape
        out["cpu_baseline"] = cpu_baseline(synth, cshape, cfg, acts)
    print(json.dumps(out))


if __name__ == "__main__":
    main()
