#!/usr/bin/env python3
"""Denoiser-step throughput of the TRACK hot path on one MI355X.

    python bench.py [--steps K] [--warmup W]     (large-model line, small model beside it)
    python bench.py [--steps K] [--warmup W] --workload small|large|long-small|long-large
    python bench.py --trajectory wan-50step|wan-50step-unipc|distilled-4step
    python bench.py --oracle-small-pair      (host oracle only, small float32 pair)

A step is one guided prediction of the video DiT (conditional and
negative-prompt branches as one batch of 2; batch 1 without guidance) plus
the fused guidance + Euler update, run through track_sample's step loop.
Inputs (weights ~N(0, 0.02) in bf16, x_T ~ N(0, 1), text ~ N(0, 1)) are
seeded synthetic stand-ins generated before the timed region and resident
in HBM.  Prints one JSON line: by default its value is the Wan-2.1-14B-shaped
model's steps/s, with the Wan-2.1-1.3B-shaped model's rate, roofline and
oracle baseline under "small" and the cost model's 50-step routed latency
from the two measured step times.  After the timed steps the library's MFMA
stream runs for ~1.7 s: "mfma_ceiling" is the sustained matrix-core rate of
this board at that moment, and each roofline carries the self-attention
kernel's fraction of it beside the fraction of the published peak.
"""
from __future__ import annotations

import argparse
import dataclasses
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "DiT denoise steps/s (large & small), MFMA util %, routed-trajectory latency"
PEAK_BF16_TFLOPS = 2500.0   # MI355X dense bf16 MFMA
PEAK_HBM_GBS = 8000.0

WORKLOADS = {
    # name: (model preset, latent preset, guidance on)
    "small": ("WAN_1_3B", "WAN_LATENT", True),
    "large": ("WAN_14B", "WAN_LATENT", True),
    "long-small": ("WAN_1_3B", "WAN_LATENT_LONG", False),
    "long-large": ("WAN_14B", "WAN_LATENT_LONG", False),
}


# HBM traffic of one self-attention launch at each step shape (B = 2,
# L = 32760; 40 heads for the large model, 12 for the small), from rocprofv3
# --pmc FETCH_SIZE and WRITE_SIZE runs, each scaled by the factor the same
# counter shows for the library's 1 GiB copy stream (2.0 and 1.0).  It
# describes the kernel source it was measured on; any other source gives null.
_ATTN_SRC = "3faf39eaf08a8839ee4f70935c8ba0e3062004095520e68d5d8fa847bf33d603"
ATTN_TRAFFIC = {"large": {"source_sha256": _ATTN_SRC, "bytes": 1.2096e10},
                "small": {"source_sha256": _ATTN_SRC, "bytes": 3.6240e9}}


def attention_source_hash():
    import hashlib
    h = hashlib.sha256()
    for f in ("attention.hip", "common.h"):
        with open(os.path.join(ROOT, "paper_2609_30096_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()


def workload_name(cfg, shape, B):
    L = shape.tokens(cfg.patch)
    size = "1.3B" if cfg.dim == 1536 else "14B"
    guid = "CFG batch 2" if B == 2 else "no CFG, batch 1"
    return (f"Wan-2.1-{size}-shaped DiT denoiser step ({cfg.blocks} blocks, d={cfg.dim}, {cfg.heads}x{cfg.head_dim} "
            f"heads, ffn {cfg.ffn_dim}), {guid}, latent {shape.channels}x{shape.frames}x{shape.height}x{shape.width} "
            f"({L} tokens), text {shape.text_len}x{cfg.text_dim}, bf16 weights/activations, fp32 residual and latent")


def step_flops(cfg, shape, B):
    """Algorithmic FLOPs of one guided prediction within a trajectory: 2MNK per GEMM, 4 B H Lq Lk dh per attention
    (the text MLP and the blocks' text keys and values, formed once per trajectory, are not counted)."""
    L = shape.tokens(cfg.patch)
    Lc, d, f, H, dh, P = shape.text_len, cfg.dim, cfg.ffn_dim, cfg.heads, cfg.head_dim, cfg.patch_elems
    M = B * L
    per_block = (2 * M * d * 3 * d + 2 * M * d * d            # QKV, self O
                 + 2 * M * d * d + 2 * M * d * d               # cross Q, cross O
                 + 2 * 2 * M * d * f                           # FFN1, FFN2
                 + 4 * B * H * L * L * dh                      # self-attention
                 + 4 * B * H * L * Lc * dh)                    # cross-attention
    rest = 2 * L * P * d + 2 * M * d * P
    return cfg.blocks * per_block + rest


def self_attn_flops(cfg, shape, B):
    L = shape.tokens(cfg.patch)
    return 4 * B * cfg.heads * L * L * cfg.head_dim


def cpu_baseline(cfg, shape, B, seed):
    """The oracle (float64 numpy) on a bounded sample of the same step, extrapolated.

    Sample: one transformer block at full width on 2048 tokens (its dense
    per-token work, after subtracting its own 2048-token attention) and the
    self-attention of 128 query rows against all L keys; the step estimate is
    blocks * B * L * (dense per token + attention per query) + head/embeddings.
    """
    import numpy as np

    from oracle import dit
    from paper_2609_30096_amd import synth

    threads = int(os.environ.get("OPENBLAS_NUM_THREADS", len(os.sched_getaffinity(0))))
    one = dataclasses.replace(cfg, blocks=1)
    params = synth.gen_params(one, seed)
    d, H, dh = cfg.dim, cfg.heads, cfg.head_dim
    L = shape.tokens(cfg.patch)
    ntok, nq = 2048, 128
    X = synth.gen_normal((9000,), (ntok, d)).astype(np.float64)
    ctx = synth.gen_text(shape, cfg.text_dim, 0, synth.BF16)
    t0 = time.perf_counter()
    ctx_emb = dit.text_embedding(params, ctx)
    e, m = dit.time_embedding(params, one, 500.0)
    t_embed = time.perf_counter() - t0
    t0 = time.perf_counter()
    dit.block(params, one, 0, X, ctx_emb, m, (1, 32, ntok // 32))
    t_block = time.perf_counter() - t0
    q = synth.gen_normal((9001,), (ntok, H, dh)).astype(np.float64)
    t0 = time.perf_counter()
    dit.attention(q, q, q)
    t_inner = time.perf_counter() - t0
    k = synth.gen_normal((9002,), (L, H, dh)).astype(np.float64)
    t0 = time.perf_counter()
    dit.attention(q[:nq], k, k)
    t_attn = time.perf_counter() - t0
    t0 = time.perf_counter()
    dit.head(params, X, e)
    t_head = time.perf_counter() - t0
    per_tok = max(t_block - t_inner, 0.0) / ntok
    per_q = t_attn / nq
    step_s = cfg.blocks * B * L * (per_tok + per_q) + B * (t_head / ntok) * L + B * t_embed
    sampled = t_embed + t_block + t_inner + t_attn + t_head
    return {
        "value": round(1.0 / step_s, 8), "unit": "steps/s", "cores": threads, "kind": "oracle",
        "sample": (f"float64 numpy oracle: 1 block at d={d} on {ntok} tokens (minus its own {ntok}-token attention) "
                   f"+ self-attention of {nq} queries vs {L} keys + head/embeddings, extrapolated to {cfg.blocks} "
                   f"blocks x batch {B} x {L} tokens; {sampled:.1f} s of CPU work measured"),
        "seconds_per_step_extrapolated": round(step_s, 1),
        "blas": "OpenBLAS (numpy)",
    }


def oracle_small_pair():
    """The oracle alone, host only: the small float32 pair (4 and 2 blocks, d = 128, 64 tokens) through a
    full calibration (M = 4 samples, N = 8 steps), top-K routing (K = 4) and a routed sample of a held-out
    seed, timed phase by phase."""
    import numpy as np

    from oracle import sampler
    from paper_2609_30096_amd import synth

    threads = int(os.environ.get("OPENBLAS_NUM_THREADS", len(os.sched_getaffinity(0))))
    cL, cS, shape, scfg = synth.TINY_LARGE, synth.TINY_SMALL, synth.TINY_LATENT, synth.TINY_SAMPLER
    large = (synth.gen_params(cL, synth.SEED_LARGE), cL)
    small = (synth.gen_params(cS, synth.SEED_SMALL), cS)
    xs = [synth.gen_latent(shape, j).astype(np.float64) for j in range(4)]
    cs = [synth.gen_text(shape, cL.text_dim, j, cL.dtype) for j in range(4)]
    u = synth.gen_null_text(shape, cL.text_dim, cL.dtype)
    t0 = time.perf_counter()
    r, q = sampler.calibrate(large, small, xs, cs, u, scfg)
    t1 = time.perf_counter()
    idx = sampler.route_topk(q, 4)
    t2 = time.perf_counter()
    x0 = sampler.sample(sampler.policy_from_indices(scfg.steps, idx), large, small,
                        synth.gen_latent(shape, 999).astype(np.float64), synth.gen_text(shape, cL.text_dim, 999, cL.dtype),
                        u, scfg)
    t3 = time.perf_counter()
    return {"metric": "oracle wall time, small float32 pair: calibrate M=4 x N=8, top-K K=4, routed sample",
            "unit": "s", "calibrate": round(t1 - t0, 3), "route": round(t2 - t1, 6), "sample": round(t3 - t2, 3),
            "cores": threads, "kind": "oracle", "small_steps": [int(i) for i in idx],
            "x0_finite": bool(np.isfinite(x0).all())}


TRAJECTORIES = {
    # name: (large preset, small preset, latent preset, sampler, calibration samples measured, of M, K)
    "wan-50step": ("WAN_14B", "WAN_1_3B", "WAN_LATENT", "WAN_SAMPLER", 1, 8, 25),
    "distilled-4step": ("WAN_14B", "WAN_1_3B", "WAN_LATENT_LONG", "DISTILLED_SAMPLER", 4, 4, 2),
    "wan-50step-unipc": ("WAN_14B", "WAN_1_3B", "WAN_LATENT", "WAN_UNIPC_SAMPLER", 1, 8, 25),
}


def trajectory(name, cal_range=None, r_out=None, r_in=None):
    """Calibration -> top-K -> routed sample for a large/small pair, timed.

    Reference-trajectory calibration runs on the first `measured` of M seeded
    samples (all M when they fit the time budget; otherwise the per-sample time
    is extrapolated to M and labelled so); top-K routes the K lowest-scoring
    steps to the small model; the routed sample and the all-large sample run on
    the held-out seed.  Also reports single-step times of each model and the
    cost model's prediction sum_i C_pi(i).

    A calibration longer than one run can hold is split over runs: with
    cal_range = (a, b) and r_out, a run calibrates samples a .. b-1 only and
    writes their scores to r_out; with r_in (those files), a run takes the
    per-sample scores from them (all M samples, each once), forms q (Eq. 5,
    sample order) and routes and samples without calibrating.
    """
    import numpy as np
    import torch

    from paper_2609_30096_amd import synth, track

    lname, sname, shname, scname, measured, M, K = TRAJECTORIES[name]
    cL, cS = getattr(synth, lname), getattr(synth, sname)
    shape, scfg = getattr(synth, shname), getattr(synth, scname)
    B = 2 if scfg.use_cfg else 1
    a0, a1 = cal_range if cal_range else (0, measured)
    if not 0 <= a0 < a1 <= M:
        raise ValueError(f"calibration samples {a0}..{a1 - 1} outside 0..{M - 1}")
    t0 = time.perf_counter()
    L = track.Model(cL, track.gen_weights_on_device(cL, synth.SEED_LARGE))
    S = track.Model(cS, track.gen_weights_on_device(cS, synth.SEED_SMALL))
    L.ensure_workspace(shape, B)
    S.ensure_workspace(shape, B)
    bf = torch.bfloat16
    cal_ids = [] if r_in else list(range(a0, a1))
    xs = [torch.from_numpy(synth.gen_latent(shape, j)).cuda() for j in cal_ids]
    cs = [torch.from_numpy(synth.gen_text(shape, cL.text_dim, j)).cuda().to(bf) for j in cal_ids]
    unc = torch.from_numpy(synth.gen_null_text(shape, cL.text_dim)).cuda().to(bf) if scfg.use_cfg else None
    x_ho = torch.from_numpy(synth.gen_latent(shape, synth.HELD_OUT)).cuda()
    c_ho = torch.from_numpy(synth.gen_text(shape, cL.text_dim, synth.HELD_OUT)).cuda().to(bf)
    torch.cuda.synchronize()
    print(f"setup {time.perf_counter() - t0:.1f} s", file=sys.stderr, flush=True)

    def timed(fn):
        torch.cuda.synchronize()
        a = time.perf_counter()
        out = fn()
        torch.cuda.synchronize()
        return out, time.perf_counter() - a

    t_start = time.perf_counter()

    def progress(j, k, n):
        if k == n - 1 or k % 10 == 9:
            who = "sample" if j < 0 else f"calibration sample {j}"
            print(f"  {who}: step {k + 1}/{n} done ({time.perf_counter() - t_start:.0f} s)", file=sys.stderr,
                  flush=True)

    track.set_progress(progress)
    one = dataclasses.replace(scfg, steps=1)
    timed(lambda: track.sample(S, None, [False], shape, one, x_ho, c_ho, unc))  # warm both
    timed(lambda: track.sample(L, None, [False], shape, one, x_ho, c_ho, unc))
    _, c_small = timed(lambda: track.sample(S, None, [False], shape, one, x_ho, c_ho, unc))
    _, c_large = timed(lambda: track.sample(L, None, [False], shape, one, x_ho, c_ho, unc))
    print(f"step: large {c_large:.3f} s, small {c_small:.3f} s", file=sys.stderr, flush=True)
    if r_in:
        # per-sample scores from earlier runs, joined in sample order
        rows, rbrows, t_cal = {}, {}, 0.0
        for path in r_in:
            with open(path) as fh:
                part = json.load(fh)
            if part["trajectory"] != name:
                raise ValueError(f"{path} holds scores of {part['trajectory']}, not {name}")
            t_cal += part["seconds"]
            for j, row, brow in zip(part["samples"], part["r"], part["band_r"]):
                rows[j], rbrows[j] = row, brow
        if sorted(rows) != list(range(M)):
            raise ValueError(f"scores for samples {sorted(rows)}; need 0..{M - 1}")
        r = np.array([rows[j] for j in range(M)], dtype=np.float64)
        rb = np.array([rbrows[j] for j in range(M)], dtype=np.float64)
        q = np.zeros(scfg.steps, dtype=np.float64)
        qb = np.zeros((scfg.steps, 6), dtype=np.float64)
        for j in range(M):  # Eq. 5, summed in sample order
            q = q + r[j]
            qb = qb + rb[j]
        q, qb = q / M, qb / M
        n_cal = M
        print(f"scores of {M} samples from {len(r_in)} file(s), {t_cal:.1f} s of calibration", file=sys.stderr,
              flush=True)
    else:
        # calibration with the frequency-band decomposition of each step's disagreement
        (r, q, rb, qb), t_cal = timed(lambda: track.calibrate(L, S, shape, xs, cs, unc, scfg, bands=True))
        n_cal = len(cal_ids)
        print(f"calibration of samples {a0}..{a1 - 1}: {t_cal:.1f} s", file=sys.stderr, flush=True)
        if r_out:
            with open(r_out, "w") as fh:
                json.dump({"trajectory": name, "samples": cal_ids, "seconds": t_cal, "r": r.tolist(),
                           "band_r": rb.tolist()}, fh)
            return {"metric": "calibration scores (partial)", "trajectory": name, "samples": cal_ids,
                    "seconds": round(t_cal, 2), "seconds_per_sample": round(t_cal / n_cal, 2), "file": r_out,
                    "step_s": {"large": round(c_large, 4), "small": round(c_small, 4)}}
    idx = track.route_policy(q, K)
    pol = np.zeros(scfg.steps, bool)
    pol[idx] = True
    x_routed, t_routed = timed(lambda: track.sample(L, S, pol, shape, scfg, x_ho, c_ho, unc))
    x_all, t_all = timed(lambda: track.sample(L, S, np.zeros(scfg.steps, bool), shape, scfg, x_ho, c_ho, unc))
    rel = float(torch.linalg.vector_norm(x_routed - x_all) / torch.linalg.vector_norm(x_all))
    # how well separated the scores are at the routing boundary: the gap between the K-th and
    # (K+1)-th smallest q against the score tolerance that per-step velocity errors of 2e-2 allow
    # (2 delta (1 + q) / (1 - delta) per step), and the narrowest gap between any two adjacent scores
    qs = np.sort(q)
    tol = lambda v: 2 * 2e-2 * (1 + v) / (1 - 2e-2)
    gaps = {"kth": round(float(qs[K - 1]), 6) if K > 0 else None,
            "k_plus_1th": round(float(qs[K]), 6) if K < len(qs) else None,
            "boundary_gap": round(float(qs[K] - qs[K - 1]), 6) if 0 < K < len(qs) else None,
            "boundary_tolerance_bf16": round(float(tol(qs[K]) + tol(qs[K - 1])), 6) if 0 < K < len(qs) else None,
            "min_adjacent_gap": round(float(np.diff(qs).min()), 6) if len(qs) > 1 else None}
    predicted = (scfg.steps - K) * c_large + K * c_small
    return {
        "metric": "routed-trajectory latency",
        "value": round(t_routed, 3),
        "unit": "s",
        "higher_is_better": False,
        "n_gpus": 1,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,0.02) bf16 weights, N(0,1) latents and text; no checkpoints)",
        "config": {"workload": f"TRACK calibration + top-K + routed sample: large {workload_name(cL, shape, B)}; "
                               f"small {cS.blocks} blocks d={cS.dim}; {scfg.steps} "
                               f"{'Euler' if scfg.solver == 'euler' else 'UniPC-%d' % scfg.order} steps, "
                               f"shift {scfg.shift}, "
                               f"{'CFG ' + str(scfg.guidance) if scfg.use_cfg else 'no CFG'}; M={M}, K={K}",
                   "steps": scfg.steps, "K": K, "M": M},
        "all_large_latency_s": round(t_all, 3),
        "speedup_vs_all_large": round(t_all / t_routed, 3),
        "cost_model_prediction_s": round(predicted, 3),
        "step_s": {"large": round(c_large, 4), "small": round(c_small, 4)},
        "steps_per_s": {"large": round(1 / c_large, 4), "small": round(1 / c_small, 4)},
        "calibration": {"samples_measured": n_cal, "seconds_measured": round(t_cal, 2),
                        "seconds_for_M": round(t_cal * M / n_cal, 1),
                        "extrapolated": n_cal != M, "q": [round(v, 5) for v in q.tolist()],
                        "band_q": {"order": ["spatial_low", "spatial_mid", "spatial_high", "temporal_low",
                                             "temporal_mid", "temporal_high"],
                                   "per_step": [[round(v, 5) for v in row] for row in qb.tolist()]},
                        "small_steps": idx.tolist(), "score_gaps": gaps},
        "routed_vs_all_large_x0_rel_l2": round(rel, 5),
        "vs_baseline": None,
    }


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--workload", choices=sorted(WORKLOADS), default=None,
                    help="time one workload only (default: the large model as the headline, the small one beside it)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--breakdown", action="store_true", help="profile one extra step per kernel class")
    ap.add_argument("--trajectory", choices=sorted(TRAJECTORIES), default=None,
                    help="time calibration, routing and a routed sample instead of single steps")
    ap.add_argument("--cal-samples", default=None, metavar="A:B",
                    help="with --trajectory and --r-out: calibrate samples A..B-1 only and save their scores")
    ap.add_argument("--r-out", default=None, help="file for the scores of a partial calibration")
    ap.add_argument("--r-in", default=None, help="comma-separated score files covering all M samples: route and "
                                                 "sample without calibrating")
    ap.add_argument("--oracle-small-pair", action="store_true",
                    help="time the host oracle alone on the small float32 pair (calibrate, route, sample)")
    args = ap.parse_args()
    if args.oracle_small_pair:
        print(json.dumps(oracle_small_pair()), flush=True)
        return

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print(f"bench.py measures one GPU only (asked for {args.gpus} GPUs, WORLD_SIZE={world}); the hot path "
              f"runs on a single GPU and is not sharded", file=sys.stderr)
        sys.exit(2)
    if args.steps < 1 or args.warmup < 0:
        ap.error("--steps must be >= 1 and --warmup >= 0")

    import numpy as np
    import torch

    from paper_2609_30096_amd import synth, track

    if not torch.cuda.is_available():
        print("bench.py needs a GPU", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)
    track.lib()

    if args.trajectory:
        cal_range = tuple(int(v) for v in args.cal_samples.split(":")) if args.cal_samples else None
        if cal_range and not args.r_out:
            ap.error("--cal-samples needs --r-out")
        r_in = args.r_in.split(",") if args.r_in else None
        print(json.dumps(trajectory(args.trajectory, cal_range, args.r_out, r_in)), flush=True)
        return

    if args.workload:
        names = [args.workload]
    else:
        names = ["large", "small"]   # the headline line: large-model steps/s, small-model steps/s beside it
    results = {}
    for name in names:
        results[name] = measure_step(name, args.steps, args.warmup, args.breakdown, not args.no_cpu_baseline)
    ceiling = sustained_mfma()
    for r in results.values():
        r["roofline"]["sustained_peak"] = ceiling["tflops"]
        r["roofline"]["frac_of_sustained"] = round(r["roofline"]["achieved"] / ceiling["tflops"], 4)
    head = results[names[0]]
    out = {
        "metric": METRIC,
        "value": head["steps_per_s"],
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": head["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic (seeded N(0,0.02) bf16 weights, N(0,1) latent and text; no checkpoints)",
        "config": head["config"],
        "mfma_util_pct": head["mfma_util_pct"],
        "step_tflop": head["step_tflop"],
        "roofline": head["roofline"],
        "output_finite": head["output_finite"],
        "board": head.get("board"),
        "mfma_ceiling": ceiling,
    }
    if "breakdown_one_step" in head:
        out["breakdown_one_step"] = head["breakdown_one_step"]
    if "cpu_baseline" in head:
        out["cpu_baseline"] = head["cpu_baseline"]
    if len(names) == 2:
        small = results[names[1]]
        out["small_steps_per_s"] = small["steps_per_s"]
        out["small"] = {k: small[k] for k in ("config", "ms_per_step", "mfma_util_pct", "step_tflop", "roofline",
                                               "output_finite", "board") if k in small}
        if "cpu_baseline" in small:
            out["small"]["cpu_baseline"] = small["cpu_baseline"]
        # the paper's cost model (total = sum_i C_pi(i)) on the measured step times, for the 50-step
        # schedule with 25 steps routed to the small model; a prediction, not a measured trajectory
        c_l, c_s = head["ms_per_step"] / 1000.0, small["ms_per_step"] / 1000.0
        out["routed_trajectory_cost_model"] = {
            "steps": 50, "small_steps": 25, "unit": "s",
            "routed_s": round(25 * c_l + 25 * c_s, 2), "all_large_s": round(50 * c_l, 2),
            "speedup": round(50 * c_l / (25 * c_l + 25 * c_s), 3),
            "kind": "sum of measured per-step times (cost model); bench.py --trajectory measures real trajectories"}
    print(json.dumps(out), flush=True)


class BoardSampler:
    """Socket power and graphics clock, read by `amd-smi metric -p -c` about once a second on a host
    thread while the timed steps run (the GPU work is untouched).  Under the MFMA-bound kernels the
    board runs at or near its power limit and below the 2.4 GHz behind the 2.5 PFLOP/s figure; this
    records the clock the timed region actually ran at.  Null where amd-smi is unavailable."""

    def __init__(self):
        self.samples, self._stop, self._th = [], False, None

    def _run(self):
        import subprocess
        while not self._stop:
            try:
                out = subprocess.run(["amd-smi", "metric", "-p", "-c", "--json"], capture_output=True, text=True,
                                     timeout=10).stdout
                g = json.loads(out)
                g = g["gpu_data"][0] if isinstance(g, dict) else g[0]
                self.samples.append((float(g["power"]["socket_power"]["value"]),
                                     float(g["clock"]["gfx_0"]["clk"]["value"])))
            except (OSError, ValueError, KeyError, IndexError, TypeError, subprocess.SubprocessError):
                pass
            time.sleep(1.0)

    def __enter__(self):
        import threading
        self._th = threading.Thread(target=self._run, daemon=True)
        self._th.start()
        return self

    def __exit__(self, *exc):
        self._stop = True
        self._th.join(timeout=15)

    def summary(self):
        kept = self.samples[1:]  # the first may precede the ramp-up
        if not kept:
            return None
        pw = sorted(x[0] for x in kept)
        ck = sorted(x[1] for x in kept)
        mhz = ck[len(ck) // 2]
        return {"socket_power_w_median": pw[len(pw) // 2], "gfx_clock_mhz_median": mhz,
                "gfx_clock_mhz_min": ck[0], "samples": len(kept),
                "bf16_mfma_peak_at_median_clock_tflops": round(256 * 4096 * mhz * 1e6 / 1e12, 1),
                "source": "amd-smi metric -p -c, once a second over the timed steps"}


def sustained_mfma(launches=24, iters=250000):
    """The sustained matrix-core rate on this board right after the timed steps: the library's MFMA stream
    (independent 16x16x32 bf16 chains on every CU, no memory traffic) on N(0,1) bf16 operands, back to
    back for about 1.7 s.  The clock under matrix work follows the operand bits, not only the power
    limit, so this is the ceiling an MFMA-bound kernel of this data can reach here; `peak` stays the
    published 2.5 PFLOP/s."""
    import torch

    from paper_2609_30096_amd import track

    ops = torch.randn(32768, device="cuda", generator=torch.Generator(device="cuda").manual_seed(0)).to(torch.bfloat16)
    sink = torch.zeros(4, device="cuda")
    track.mfma_stream(ops, iters, sink)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    flop = sum(track.mfma_stream(ops, iters, sink) for _ in range(launches))
    e1.record()
    torch.cuda.synchronize()
    tflops = flop / e0.elapsed_time(e1) / 1e9
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return {"tflops": round(tflops, 1), "frac_of_published_peak": round(tflops / PEAK_BF16_TFLOPS, 4),
            "clock_mhz_at_full_issue": round(tflops * 1e12 / (cus * 4096) / 1e6),
            "launches": launches, "seconds": round(e0.elapsed_time(e1) / 1000.0, 2),
            "kernel": "mfma_stream_kernel (track_mfma_stream), N(0,1) bf16 operands"}


def measure_step(name, steps, warmup, breakdown_on, with_cpu):
    """Time `steps` routed-sampler steps of one workload (after `warmup` untimed steps)."""
    import numpy as np
    import torch

    from paper_2609_30096_amd import synth, track

    mname, sname, use_cfg = WORKLOADS[name]
    cfg = getattr(synth, mname)
    shape = getattr(synth, sname)
    B = 2 if use_cfg else 1
    seed = synth.SEED_SMALL if cfg.dim == 1536 else synth.SEED_LARGE

    t_setup = time.perf_counter()
    model = track.Model(cfg, track.gen_weights_on_device(cfg, seed))
    x_T = torch.from_numpy(synth.gen_latent(shape, synth.HELD_OUT)).cuda()
    cond = torch.from_numpy(synth.gen_text(shape, cfg.text_dim, synth.HELD_OUT)).cuda().to(torch.bfloat16)
    unc = torch.from_numpy(synth.gen_null_text(shape, cfg.text_dim)).cuda().to(torch.bfloat16) if use_cfg else None
    model.ensure_workspace(shape, B)
    torch.cuda.synchronize()
    print(f"[{name}] setup {time.perf_counter() - t_setup:.1f} s: {cfg.n_params() / 1e9:.2f} B params, "
          f"workspace {model.workspace.numel() / 2**30:.2f} GiB", file=sys.stderr, flush=True)

    def run(n):
        scfg = synth.SamplerConfig(steps=n, shift=5.0, guidance=5.0, use_cfg=use_cfg)
        return track.sample(model, None, np.zeros(n, bool), shape, scfg, x_T, cond, unc)

    if warmup:
        run(warmup)
        torch.cuda.synchronize()
        print(f"[{name}] warmup done", file=sys.stderr, flush=True)

    track.profile_reset()
    track.profile_enable([track.PROF_ATTN_SELF])
    torch.cuda.synchronize()
    with BoardSampler() as board:
        t0 = time.perf_counter()
        x0 = run(steps)
        torch.cuda.synchronize()
        elapsed = time.perf_counter() - t0
    track.profile_enable([])
    n_attn, attn_ms = track.profile_read(track.PROF_ATTN_SELF)
    finite = bool(torch.isfinite(x0).all().item())
    print(f"[{name}] timed {steps} steps in {elapsed:.3f} s; x0 finite: {finite}", file=sys.stderr, flush=True)

    res = {}
    if breakdown_on:
        track.profile_reset()
        track.profile_enable()
        run(1)
        track.profile_enable([])
        names = ["attn_self", "attn_cross", "gemm", "norm", "step", "other"]
        bd = {}
        for k, nm in enumerate(names):
            n, ms = track.profile_read(k)
            bd[nm] = {"launches": n, "ms": round(ms, 3)}
        res["breakdown_one_step"] = bd
    model.close()
    del model, x0
    torch.cuda.empty_cache()

    ms_per_step = 1000.0 * elapsed / steps
    flops = step_flops(cfg, shape, B)
    attn_flops = self_attn_flops(cfg, shape, B)
    avg_attn_s = attn_ms / 1000.0 / max(n_attn, 1)
    achieved = attn_flops / avg_attn_s / 1e12
    traffic = ATTN_TRAFFIC.get(name)
    res.update({
        "steps_per_s": round(steps / elapsed, 5),
        "ms_per_step": round(ms_per_step, 3),
        "config": {"workload": workload_name(cfg, shape, B), "batch": B, "tokens": shape.tokens(cfg.patch),
                   "blocks": cfg.blocks, "dim": cfg.dim, "heads": cfg.heads, "ffn_dim": cfg.ffn_dim,
                   "text_len": shape.text_len, "parallelism": "single GPU"},
        "mfma_util_pct": round(100.0 * flops / (ms_per_step / 1000.0) / (PEAK_BF16_TFLOPS * 1e12), 2),
        "step_tflop": round(flops / 1e12, 2),
        "roofline": {
            "kernel": "flash_attn_bf16_kernel (3D self-attention)",
            "bound": "mfma",
            "achieved": round(achieved, 1),
            "peak": PEAK_BF16_TFLOPS,
            "unit": "TFLOP/s",
            "frac": round(achieved / PEAK_BF16_TFLOPS, 4),
            "traffic": (traffic["bytes"] if traffic and traffic["source_sha256"] == attention_source_hash()
                        else None),
            "traffic_unit": "bytes per launch (HBM fetch + write)",
            "launches": n_attn,
            "avg_launch_ms": round(1000.0 * avg_attn_s, 3),
            "flop_per_launch": attn_flops,
        },
        "output_finite": finite,
        "board": board.summary(),
    })
    if with_cpu:
        print(f"[{name}] cpu baseline (oracle) ...", file=sys.stderr, flush=True)
        res["cpu_baseline"] = cpu_baseline(cfg, shape, B, seed)
    return res


if __name__ == "__main__":
    main()
