"""Performance cases of the TRACK denoising path on one MI355X.

Each case is one call (or one short chain of calls) a program makes through
``paper_2609_30096_amd.track``: a whole calibration or guided prediction, one
full-width transformer block, or one of the component entry points (a
projection, attention, the norms, the band decomposition).  Sizes are the
library's own workloads: the Wan-2.1 1.3B and 14B widths on the 81-frame
480 x 832 video latent (16 x 21 x 60 x 104, 32760 tokens), the same frame size
as a single image (16 x 1 x 60 x 104, 1560 tokens), the 512-token text context
and the small float32 pair.  ``draw`` spreads the same calls over their ranges,
ragged sizes included.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_30096_amd import synth, track

EPI = {"bias": track.EPI_BIAS, "gelu": track.EPI_BIAS_GELU, "gate": track.EPI_GATE_RESID,
       "resid": track.EPI_RESID, "f32": track.EPI_BIAS_F32}
LOG2E = 1.4426950408889634
MAX_FLOPS = 8.0e13  # no drawn case costs more than block_14b_video


# ---------------------------------------------------------------- the cases
def _model(blocks, heads, head_dim, ffn, text_dim, dtype):
    return {"blocks": blocks, "heads": heads, "head_dim": head_dim, "ffn": ffn, "text_dim": text_dim, "dtype": dtype}


def _latent(frames, height, width, text_len):
    return {"frames": frames, "height": height, "width": width, "text_len": text_len}


def listed():
    return [
        # The smallest whole call: calibration of the small float32 pair (4 and
        # 2 blocks, width 128, 64 tokens), four samples of eight guided steps;
        # every kernel is tiny, so launches and latency count.
        {"name": "calibrate_small_f32", "kind": "calibrate", **_model(4, 4, 32, 512, 128, "f32"),
         **_latent(4, 8, 8, 16), "small_blocks": 2, "samples": 4, "steps": 8, "cfg": True},
        # One guided prediction of the full 30-block 1.3B model on a single
        # frame: what a text-to-image step or a preview costs.
        {"name": "forward_13b_image", "kind": "forward", **_model(30, 12, 128, 8960, 4096, "bf16"),
         **_latent(1, 60, 104, 512), "cfg": True},
        # The headline workload's unit: one 14B-wide block on the video latent
        # with guidance (one fortieth of a denoising step, and its embeddings
        # and head).
        {"name": "block_14b_video", "kind": "forward", **_model(1, 40, 128, 13824, 4096, "bf16"),
         **_latent(21, 60, 104, 512), "cfg": True},
        # Projections: the widest of the 14B video step, the gated float32
        # residual update of the 1.3B video step (memory bound as much as
        # matrix bound), and the text keys / values of every block, a small one.
        {"name": "linear_14b_ffn1", "kind": "linear", "dtype": "bf16", "epi": "gelu", "M": 65520, "N": 13824, "K": 5120},
        {"name": "linear_13b_o", "kind": "linear", "dtype": "bf16", "epi": "gate", "M": 65520, "N": 1536, "K": 1536},
        {"name": "linear_13b_text_kv", "kind": "linear", "dtype": "bf16", "epi": "bias", "M": 1024, "N": 3072, "K": 1536},
        # Attention: the 1.3B video step's self-attention (q pre-scaled, as the
        # forward passes it), the single image's on plain q, and the video's
        # cross-attention over the text.
        {"name": "attn_13b_video", "kind": "attention", "dtype": "bf16", "B": 2, "heads": 12, "head_dim": 128,
         "Lq": 32760, "Lk": 32760, "q_log2": True},
        {"name": "attn_13b_image", "kind": "attention", "dtype": "bf16", "B": 2, "heads": 12, "head_dim": 128,
         "Lq": 1560, "Lk": 1560, "q_log2": False},
        {"name": "attn_13b_text", "kind": "attention", "dtype": "bf16", "B": 2, "heads": 12, "head_dim": 128,
         "Lq": 32760, "Lk": 512, "q_log2": True},
        # Norms: the modulated LayerNorm of the single image, and the fused
        # q / k RMSNorm with 3D RoPE of the 14B video step (in place).
        {"name": "layernorm_13b_image", "kind": "layernorm", "dtype": "bf16", "rows": 3120, "d": 1536, "mod": True},
        {"name": "norm_rope_14b_video", "kind": "norm_rope", "dtype": "bf16", "B": 2, "heads": 40, "head_dim": 128,
         "grid_f": 21, "grid_h": 30, "grid_w": 52},
        # The band decomposition that a calibration with band scores runs at
        # every step, on the video latent with guidance.
        {"name": "bands_video", "kind": "bands", "frames": 21, "height": 60, "width": 104, "B": 2},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["calibrate", "forward", "forward", "linear", "linear", "linear", "attention", "attention",
                       "attention", "layernorm", "norm_rope", "bands"])
    if kind == "calibrate":
        # small float32 pairs: the parity configuration's neighbourhood
        hd = rng.choice([32, 64, 128])
        return {"kind": kind, **_model(rng.randint(2, 4), rng.randint(2, 4), hd, 64 * rng.randint(3, 10), 128, "f32"),
                **_latent(rng.randint(1, 4), 2 * rng.randint(3, 7), 2 * rng.randint(3, 7), rng.randint(7, 32)),
                "small_blocks": 1, "samples": rng.randint(1, 4), "steps": rng.randint(2, 8),
                "cfg": rng.random() < 0.7}
    if kind == "forward":
        # bfloat16 models up to the 1.3B width and some way beyond
        heads = rng.choice([3, 5, 6, 8, 10, 12, 16, 20])
        return {"kind": kind, **_model(rng.randint(1, 4), heads, 128, 64 * _log(rng, 2 * heads, 12 * heads),
                                       64 * rng.randint(8, 64), "bf16"),
                **_latent(rng.choice([1, 1, 3, 5, 9, 13, 21]), 2 * _log(rng, 6, 45), 2 * _log(rng, 6, 80),
                          rng.choice([512, 512, 226, 77, 333])),
                "cfg": rng.random() < 0.6}
    if kind == "linear":
        heads = rng.choice([3, 6, 8, 9, 12, 12, 16, 24, 40, 40])
        d = 128 * heads
        f = 64 * rng.randint(4 * heads, 12 * heads)
        role = rng.choice(["qk", "v", "o", "co", "ffn1", "ffn2", "head", "embed"])
        n, k, epi = {"qk": (2 * d, d, "bias"), "v": (d, d, "bias"), "o": (d, d, "gate"), "co": (d, d, "resid"),
                     "ffn1": (f, d, "gelu"), "ffn2": (d, f, "gate"), "head": (64, d, "f32"),
                     "embed": (d, 64, "f32")}[role]
        m = _log(rng, 100, 65520)
        return {"kind": kind, "dtype": "bf16", "epi": epi, "M": m, "N": n, "K": k}
    if kind == "attention":
        if rng.random() < 0.2:
            lq = _log(rng, 32, 1500)
            return {"kind": kind, "dtype": "f32", "B": rng.randint(1, 2), "heads": rng.randint(2, 8),
                    "head_dim": rng.choice([32, 64, 128]), "Lq": lq,
                    "Lk": rng.choice([lq, rng.randint(8, 512)]), "q_log2": False}
        lq = _log(rng, 128, 32760)
        lk = lq if rng.random() < 0.65 else rng.choice([512, rng.randint(16, 512)])
        return {"kind": kind, "dtype": "bf16", "B": rng.randint(1, 2), "heads": rng.choice([3, 8, 12, 12, 24, 40]),
                "head_dim": 128, "Lq": lq, "Lk": lk, "q_log2": rng.random() < 0.6}
    if kind == "layernorm":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "rows": _log(rng, 64, 65520),
                "d": 128 * rng.choice([2, 3, 8, 12, 12, 20, 40]), "mod": rng.random() < 0.7}
    if kind == "norm_rope":
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "B": rng.randint(1, 2),
                "heads": rng.choice([2, 5, 12, 12, 24, 40]), "head_dim": 128, "grid_f": rng.choice([1, 3, 9, 21]),
                "grid_h": _log(rng, 5, 45), "grid_w": _log(rng, 5, 80)}
    return {"kind": "bands", "frames": rng.choice([1, 5, 13, 21, 33]), "height": 2 * _log(rng, 8, 45),
            "width": 2 * _log(rng, 8, 80), "B": rng.randint(1, 2)}


def draw(rng):
    while True:
        c = _draw_once(rng)
        if work(c)["flops"] <= MAX_FLOPS:
            return c


# ---------------------------------------------------------------- inputs
def _dt(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _code(case):
    return track.DTYPE_BF16 if case["dtype"] == "bf16" else track.DTYPE_F32


def _gen(seed, salt=0):
    return torch.Generator(device="cuda").manual_seed(1000003 * seed + salt)


def _randn(g, *shape, scale=1.0, dtype=torch.float32):
    t = torch.empty(shape, device="cuda", dtype=torch.float32).normal_(generator=g)
    return (t.mul_(scale) if scale != 1.0 else t).to(dtype)


def _dit(case, blocks=None):
    d = case["heads"] * case["head_dim"]
    return synth.DiTConfig(blocks=case["blocks"] if blocks is None else blocks, dim=d, heads=case["heads"],
                           head_dim=case["head_dim"], ffn_dim=case["ffn"], text_dim=case["text_dim"],
                           dtype=synth.BF16 if case["dtype"] == "bf16" else synth.F32)


def _shape(case):
    return synth.LatentShape(16, case["frames"], case["height"], case["width"], case["text_len"])


def _weights(cfg, g):
    """A weight buffer in the library's layout and name -> view of it: N(0, 0.02)
    weights, biases and modulation tables, gains around one."""
    table, total = track.weight_table(cfg)
    buf = torch.empty(total, dtype=torch.uint8, device="cuda")
    dt = torch.bfloat16 if cfg.dtype == synth.BF16 else torch.float32
    size = 2 if cfg.dtype == synth.BF16 else 4
    views = {}
    for name, shape, off in table:
        n = int(np.prod(shape))
        v = buf[off:off + n * size].view(dt).view(shape)
        if "norm_" in name:
            v.copy_(_randn(g, *shape, scale=0.1) + 1.0)
        else:
            v.copy_(_randn(g, *shape, scale=0.02))
        views[name] = v
    return buf, views


def _text(case, g):
    return _randn(g, case["text_len"], case["text_dim"], dtype=_dt(case))


def _x(case, g):
    return _randn(g, 16, case["frames"], case["height"], case["width"])


def _inputs(case, seed):
    """The plain tensors of a case, from the seed alone."""
    g = _gen(seed)
    k = case["kind"]
    if k == "calibrate":
        large = _weights(_dit(case), g)
        small = _weights(_dit(case, case["small_blocks"]), g)
        xs = [_x(case, g) for _ in range(case["samples"])]
        conds = [_text(case, g) for _ in range(case["samples"])]
        return {"large": large, "small": small, "x": xs, "cond": conds,
                "uncond": _text(case, g) if case["cfg"] else None}
    if k == "forward":
        w = _weights(_dit(case), g)
        return {"w": w, "x": _x(case, g), "cond": _text(case, g), "uncond": _text(case, g) if case["cfg"] else None}
    if k == "linear":
        dt = _dt(case)
        m, n, kk = case["M"], case["N"], case["K"]
        s = {"A": _randn(g, m, kk, dtype=dt), "W": _randn(g, n, kk, scale=0.02, dtype=dt),
             "bias": _randn(g, n, scale=0.02, dtype=dt)}
        if case["epi"] == "gate":
            s["gate"] = _randn(g, n, scale=0.5)
        if case["epi"] in ("gate", "resid"):
            s["out"] = _randn(g, m, n)
        return s
    if k == "attention":
        dt = _dt(case)
        B, H, dh, lq, lk = case["B"], case["heads"], case["head_dim"], case["Lq"], case["Lk"]
        ldv = (lk + 63) // 64 * 64
        # q and k as the RMSNorms leave them, v as a projection of normalised rows
        scale = LOG2E / math.sqrt(dh) if case["q_log2"] else 1.0
        vt = torch.zeros(B, H, dh, ldv, device="cuda", dtype=dt)
        s = {"q": _randn(g, B * lq, H * dh, scale=scale, dtype=dt), "k": _randn(g, B * lk, H * dh, dtype=dt), "vt": vt}
        vt[..., :lk] = _randn(g, B, H, dh, lk, scale=0.8, dtype=dt)
        return s
    if k == "layernorm":
        d = case["d"]
        x = _randn(g, case["rows"], d, scale=2.0) + _randn(g, case["rows"], 1)
        s = {"x": x, "scale": None, "shift": None}
        if case["mod"]:
            s["scale"], s["shift"] = _randn(g, d, scale=0.1), _randn(g, d, scale=0.1)
        return s
    if k == "norm_rope":
        d = case["heads"] * case["head_dim"]
        rows = case["B"] * case["grid_f"] * case["grid_h"] * case["grid_w"]
        dt = _dt(case)
        # the q, k, v rows of the fused projection buffer
        return {"buf": _randn(g, rows, 3 * d, scale=1.3, dtype=dt), "gq": (_randn(g, d, scale=0.1) + 1.0).to(dt),
                "gk": (_randn(g, d, scale=0.1) + 1.0).to(dt)}
    n = 16 * case["frames"] * case["height"] * case["width"]
    base = _randn(g, case["B"] * n)
    return {"L": base, "S": base + _randn(g, case["B"] * n, scale=0.2)}


def prepare(case, seed):
    s = _inputs(case, seed)
    k = case["kind"]
    st = {"case": case, **s}
    if k in ("calibrate", "forward"):
        B = 2 if case["cfg"] else 1
        st["shape"] = _shape(case)
        names = ("large", "small") if k == "calibrate" else ("w",)
        for name in names:
            cfg = _dit(case, case["small_blocks"] if name == "small" else None)
            m = track.Model(cfg, s[name][0])
            m.ensure_workspace(st["shape"], B)
            st[name] = m
        if k == "calibrate":
            st["sampler"] = synth.SamplerConfig(steps=case["steps"], shift=3.0, guidance=5.0, use_cfg=case["cfg"])
    elif k == "linear" and "out" not in st:
        dt = torch.float32 if case["epi"] == "f32" else _dt(case)
        st["out"] = torch.empty(case["M"], case["N"], device="cuda", dtype=dt)
    elif k == "attention":
        st["out"] = torch.empty(case["B"] * case["Lq"], case["heads"] * case["head_dim"], device="cuda", dtype=_dt(case))
    elif k == "layernorm":
        st["y"] = torch.empty(case["rows"], case["d"], device="cuda", dtype=_dt(case))
    elif k == "bands":
        st["shape"] = synth.LatentShape(16, case["frames"], case["height"], case["width"], 512)
        st["ws"] = torch.empty(track.band_workspace_bytes(st["shape"]), device="cuda", dtype=torch.uint8)
    return st


# ---------------------------------------------------------------- one pass
T_STEP = 620.0   # a mid-trajectory model timestep
GUIDANCE = 5.0


def run(st):
    case = st["case"]
    k = case["kind"]
    if k == "calibrate":
        r, q, x0 = track.calibrate(st["large"], st["small"], st["shape"], st["x"], st["cond"], st["uncond"],
                                   st["sampler"], return_x0=True)
        return {"r": r, "q": q, "x0": x0}
    if k == "forward":
        return track.dit_forward(st["w"], st["shape"], st["x"], T_STEP, st["cond"], st["uncond"], GUIDANCE)
    if k == "linear":
        track.op_linear(_code(case), EPI[case["epi"]], st["A"], st["W"], st["bias"], st["out"], gate=st.get("gate"))
        return st["out"]
    if k == "attention":
        w = case["heads"] * case["head_dim"]
        track.op_attention(_code(case), case["B"], case["heads"], case["head_dim"], case["Lq"], case["Lk"], st["q"], w,
                           st["k"], w, st["vt"], st["vt"].shape[-1], st["out"], w, q_log2=case["q_log2"])
        return st["out"]
    if k == "layernorm":
        track.op_layernorm(_code(case), st["x"], st["y"], st["scale"], st["shift"])
        return st["y"]
    if k == "norm_rope":
        track.op_rmsnorm_rope_qk(_code(case), st["buf"], case["heads"], case["head_dim"], st["gq"], st["gk"],
                                 grid=(case["grid_f"], case["grid_h"], case["grid_w"]))
        return st["buf"]
    return track.op_band_energy(st["shape"], case["B"], GUIDANCE, st["L"], st["S"], st["ws"])


# ---------------------------------------------------------------- the work a pass cannot do without
def _forward_work(case, blocks):
    d, f, td = case["heads"] * case["head_dim"], case["ffn"], case["text_dim"]
    B = 2 if case["cfg"] else 1
    L = case["frames"] * (case["height"] // 2) * (case["width"] // 2)
    lc = case["text_len"]
    # per row of tokens: q, k, v, o, cross q, cross o, the MLP; per text row: keys and values
    block = 2 * B * L * (6 * d * d + 2 * d * f) + 2 * B * lc * 2 * d * d + 4 * B * L * (L + lc) * d
    flops = blocks * block + 2 * L * 64 * d + 2 * B * L * 64 * d + 2 * B * lc * (td * d + d * d) + 2 * (256 * d + 7 * d * d)
    size = 2 if case["dtype"] == "bf16" else 4
    params = blocks * (8 * d * d + 2 * d * f) + 128 * d + 256 * d + 7 * d * d + td * d + d * d
    nbytes = params * size + 2 * 16 * case["frames"] * case["height"] * case["width"] * 4 + B * lc * td * size
    return flops, nbytes


def work(case):
    k = case["kind"]
    size = 2 if case.get("dtype") == "bf16" else 4
    if k == "calibrate":
        fl, bl = _forward_work(case, case["blocks"])
        fs, bs = _forward_work(case, case["small_blocks"])
        n = case["samples"] * case["steps"]
        return {"bytes": bl + bs, "flops": n * (fl + fs)}
    if k == "forward":
        fl, by = _forward_work(case, case["blocks"])
        return {"bytes": by, "flops": fl}
    if k == "linear":
        m, n, kk = case["M"], case["N"], case["K"]
        out = {"bias": size, "gelu": size, "f32": 4, "gate": 8, "resid": 8}[case["epi"]]
        return {"bytes": (m * kk + n * kk) * size + m * n * out, "flops": 2 * m * n * kk}
    if k == "attention":
        B, w, lq, lk = case["B"], case["heads"] * case["head_dim"], case["Lq"], case["Lk"]
        return {"bytes": 2 * B * (lq + lk) * w * size, "flops": 4 * B * w * lq * lk}
    if k == "layernorm":
        n = case["rows"] * case["d"]
        return {"bytes": n * (4 + size), "flops": 8 * n}
    if k == "norm_rope":
        n = case["B"] * case["grid_f"] * case["grid_h"] * case["grid_w"] * 2 * case["heads"] * case["head_dim"]
        return {"bytes": 2 * n * size, "flops": 8 * n}
    # the transforms as fast ones: 5 n log2 n complex, half of it for real input
    n = 16 * case["frames"] * case["height"] * case["width"]
    logs = math.log2(case["height"]) + math.log2(case["width"]) + math.log2(max(2, case["frames"]))
    return {"bytes": 2 * case["B"] * n * 4, "flops": int(2.5 * n * logs)}


# Relative 2-norms.  Each is about four times the largest error against the
# float64 results over the listed and drawn cases, rounded up: bfloat16 outputs
# round at 2^-9 (1.7e-3 measured); attention also rounds its probabilities
# (2.4e-3); a guided bfloat16 prediction amplifies each branch's rounding by the
# guidance scale (1.3e-2, 2.3e-3 without guidance); float32 sums of up to 28736
# terms stay below 1e-6, the others below 4e-7 (attention) and 2e-7.
def tolerance(case):
    k = case["kind"]
    bf = case.get("dtype") == "bf16"
    if k == "calibrate":
        return {"rel": 2e-6}
    if k == "forward":
        return {"rel": 5e-2 if case["cfg"] else 1e-2}
    if k == "linear":
        return {"rel": 6e-3 if case["epi"] in ("bias", "gelu") else 5e-6}
    if k == "attention":
        return {"rel": 1e-2 if bf else 2e-6}
    if k in ("layernorm", "norm_rope"):
        return {"rel": 6e-3 if bf else 1e-6}
    return {"rel": 1e-6}


# ---------------------------------------------------------------- float64 results
def _f64(t):
    return t.to(torch.float64)


def _ln64(x):
    xc = x - x.mean(-1, keepdim=True)
    return xc / torch.sqrt((xc * xc).mean(-1, keepdim=True) + 1e-6)


def _rms64(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6) * g


def _gelu64(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _rope64(x, grid):
    """x [L, heads, dh]: pairs (2i, 2i+1) turned by pos * 10000^(-2i/n) per section."""
    L, H, dh = x.shape
    ds = 2 * (dh // 6)
    pos = torch.meshgrid(*[torch.arange(e, device=x.device, dtype=torch.float64) for e in grid], indexing="ij")
    ang = []
    for p, n in zip(pos, (dh - 2 * ds, ds, ds)):
        w = 10000.0 ** (-2.0 * torch.arange(n // 2, device=x.device, dtype=torch.float64) / n)
        ang.append(p.reshape(-1, 1) * w)
    ang = torch.cat(ang, 1)[:, None, :]
    a, b = x[..., 0::2], x[..., 1::2]
    c, s = torch.cos(ang), torch.sin(ang)
    return torch.stack([a * c - b * s, a * s + b * c], -1).reshape(L, H, dh)


def _attn64(q, k, v, scale):
    """q [Lq, H, dh], k, v [Lk, H, dh] -> [Lq, H * dh]; rows in pieces that bound the logits' memory."""
    lq, H, dh = q.shape
    out = torch.empty(lq, H, dh, device=q.device, dtype=torch.float64)
    step = max(64, int(2e8) // max(1, k.shape[0]))
    for h in range(H):
        kt, vh = k[:, h].t().contiguous(), v[:, h].contiguous()
        for r in range(0, lq, step):
            p = torch.softmax(q[r:r + step, h].contiguous() @ kt * scale, -1)
            out[r:r + step, h] = p @ vh
    return out.reshape(lq, H * dh)


def _forward64(p, case, blocks, x, t, ctx):
    """One branch of the denoiser, latent in and velocity out, in float64."""
    H, dh = case["heads"], case["head_dim"]
    d = H * dh
    C, F, Hh, Ww = x.shape
    grid = (F, Hh // 2, Ww // 2)
    L = grid[0] * grid[1] * grid[2]

    def lin(v, name, w=".w", b=".b"):
        return v @ _f64(p[name + w]).t() + _f64(p[name + b])

    def heads(v):
        return v.reshape(-1, H, dh)

    tok = _f64(x).reshape(C, F, Hh // 2, 2, Ww // 2, 2).permute(1, 2, 4, 0, 3, 5).reshape(L, C * 4)
    X = lin(tok, "patch")
    half = 128
    ang = t * 10000.0 ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    s = torch.cat([torch.cos(ang), torch.sin(ang)])
    silu = torch.nn.functional.silu
    e = lin(silu(lin(s, "time", ".w1", ".b1")), "time", ".w2", ".b2")
    m = lin(silu(e), "mod").reshape(6, d)
    c = lin(_gelu64(lin(_f64(ctx), "text", ".w1", ".b1")), "text", ".w2", ".b2")
    scale = 1.0 / math.sqrt(dh)
    for b in range(blocks):
        n = f"blk{b}."
        sh1, sc1, g1, sh2, sc2, g2 = m + _f64(p[n + "mod"])
        qkv = lin(_ln64(X) * (1.0 + sc1) + sh1, n + "qkv")
        q = _rope64(heads(_rms64(qkv[:, :d], _f64(p[n + "norm_q"]))), grid)
        k = _rope64(heads(_rms64(qkv[:, d:2 * d], _f64(p[n + "norm_k"]))), grid)
        X = X + g1 * lin(_attn64(q, k, heads(qkv[:, 2 * d:]), scale), n + "o")
        q = heads(_rms64(lin(_ln64(X), n + "cq"), _f64(p[n + "norm_cq"])))
        kv = lin(c, n + "ckv")
        k = heads(_rms64(kv[:, :d], _f64(p[n + "norm_ck"])))
        X = X + lin(_attn64(q, k, heads(kv[:, d:]), scale), n + "co")
        hid = _gelu64(lin(_ln64(X) * (1.0 + sc2) + sh2, n + "ffn1"))
        X = X + g2 * lin(hid, n + "ffn2")
    sh, sc = _f64(p["head.mod"]) + e
    out = lin(_ln64(X) * (1.0 + sc) + sh, "head")
    return out.reshape(*grid, C, 2, 2).permute(3, 0, 1, 4, 2, 5).reshape(C, F, Hh, Ww)


def _guided64(p, case, blocks, x, t, cond, uncond):
    c = _forward64(p, case, blocks, x, t, cond)
    if uncond is None:
        return c
    u = _forward64(p, case, blocks, x, t, uncond)
    return u + GUIDANCE * (c - u)


def exact(case, seed):
    k = case["kind"]
    s = _inputs(case, seed)
    if k == "calibrate":
        N, M = case["steps"], case["samples"]
        u = [1.0 - i / N for i in range(N + 1)]
        sig = [3.0 * v / (1.0 + 2.0 * v) for v in u]
        r = np.zeros((M, N))
        x0 = []
        for j in range(M):
            x = _f64(s["x"][j])
            for i in range(N):
                pl = _guided64(s["large"][1], case, case["blocks"], x, 1000.0 * sig[i], s["cond"][j], s["uncond"])
                ps = _guided64(s["small"][1], case, case["small_blocks"], x, 1000.0 * sig[i], s["cond"][j], s["uncond"])
                r[j, i] = float((ps - pl).norm() / pl.norm())
                x = x + (sig[i + 1] - sig[i]) * pl
            x0.append(x)
        return {"r": r, "q": r.mean(0), "x0": x0}
    if k == "forward":
        return _guided64(s["w"][1], case, case["blocks"], s["x"], T_STEP, s["cond"], s["uncond"])
    if k == "linear":
        w = _f64(s["W"]).t().contiguous()
        b = _f64(s["bias"])
        out = torch.empty(case["M"], case["N"], device="cuda", dtype=torch.float64)
        for r in range(0, case["M"], 8192):
            v = _f64(s["A"][r:r + 8192]) @ w + b
            if case["epi"] == "gelu":
                v = _gelu64(v)
            elif case["epi"] == "gate":
                v = _f64(s["out"][r:r + 8192]) + _f64(s["gate"]) * v
            elif case["epi"] == "resid":
                v = _f64(s["out"][r:r + 8192]) + v
            out[r:r + 8192] = v
        return out
    if k == "attention":
        B, H, dh, lq, lk = case["B"], case["heads"], case["head_dim"], case["Lq"], case["Lk"]
        scale = math.log(2.0) if case["q_log2"] else 1.0 / math.sqrt(dh)
        outs = []
        for b in range(B):
            v = _f64(s["vt"][b, :, :, :lk]).permute(2, 0, 1)
            outs.append(_attn64(_f64(s["q"][b * lq:(b + 1) * lq]).view(lq, H, dh),
                                _f64(s["k"][b * lk:(b + 1) * lk]).view(lk, H, dh), v, scale))
        return torch.cat(outs)
    if k == "layernorm":
        y = _ln64(_f64(s["x"]))
        return y * (1.0 + _f64(s["scale"])) + _f64(s["shift"]) if case["mod"] else y
    if k == "norm_rope":
        H, dh = case["heads"], case["head_dim"]
        d = H * dh
        grid = (case["grid_f"], case["grid_h"], case["grid_w"])
        L = grid[0] * grid[1] * grid[2]
        out = _f64(s["buf"])
        for seg, g in ((0, s["gq"]), (1, s["gk"])):
            for b in range(case["B"]):
                v = _rms64(out[b * L:(b + 1) * L, seg * d:(seg + 1) * d], _f64(g))
                out[b * L:(b + 1) * L, seg * d:(seg + 1) * d] = _rope64(v.reshape(L, H, dh), grid).reshape(L, d)
        return out
    # band energies of the guided difference on the C x F x H x W latent
    F, Hh, Ww, B = case["frames"], case["height"], case["width"], case["B"]
    n = 16 * F * Hh * Ww

    def guided(v):
        v = _f64(v)
        p = v[n:] + GUIDANCE * (v[:n] - v[n:]) if B == 2 else v
        return p.view(F, Hh // 2, Ww // 2, 16, 2, 2).permute(3, 0, 1, 4, 2, 5).reshape(16, F, Hh, Ww)

    diff = guided(s["S"]) - guided(s["L"])

    def fold(m):
        a = np.arange(m)
        return np.minimum(a, m - a).astype(np.int64)

    e2 = (torch.fft.fft2(diff, norm="ortho").abs() ** 2).sum((0, 1)).cpu().numpy()
    e1 = (torch.fft.fft(diff, dim=1, norm="ortho").abs() ** 2).sum((0, 2, 3)).cpu().numpy()
    rad = (fold(Hh)[:, None] * Ww) ** 2 + (fold(Ww)[None, :] * Hh) ** 2
    hw2 = (Hh * Ww) ** 2
    sb = np.where(36 * rad < hw2, 0, np.where(9 * rad < hw2, 1, 2))
    a = fold(F)
    tb = np.where(6 * a < F, 0, np.where(3 * a < F, 1, 2))
    return np.array([e2[sb == i].sum() for i in range(3)] + [e1[tb == i].sum() for i in range(3)])
