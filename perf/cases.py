"""The measured workloads of the block-wise causal attention library.

A case is a dict of plain values.  `kind` says which of the library's call sequences a pass is:

  forward   the whole sequence attended once, no cache           Attention.forward
  train     the attention's share of a training step             Attention.forward_lse, Attention.backward
  step      one cached step: write the new frames' K/V, attend   nfd_kvcache_append_attn_fwd
  rope      one cached step of a model with 3D rotary positions; Attention.rope_append, Attention.forward
            `drop` > 0: the window slides first                  nfd_kvcache_shift before them
  rope8     the same over the 8-bit KV cache                     nfd_kvcache_shift_fp8, nfd_rope_kvcache_append_fp8,
                                                                 nfd_block_causal_attn_fwd_fp8kv

B, H, D: batch, heads, head width; T tokens a frame (gh x gw of the latent grid); kv frames of keys once the new ones are
written, of which the last n are the queries; F frames of cache capacity.
"""
import math

import torch

from paper_2506_01380_amd import binding as nb

SECTIONS = (16, 24, 24)  # head features that follow time, grid row and grid column
FP8_SCALE = 6.0 / 448.0  # six sigma of the inputs at the top of the E4M3 range


def _case(name, kind, dtype, B, H, gh, gw, kv, n, F=None, drop=0, D=64):
    return dict(name=name, kind=kind, dtype=dtype, B=B, H=H, D=D, gh=gh, gw=gw, T=gh * gw, kv=kv, n=n, F=F or kv, drop=drop)


def listed():
    return [
        # the smallest call: a unit test or a demonstration in full precision; nothing but latency
        _case("tiny_fp32", "forward", "fp32", 1, 2, 4, 4, 4, 4),
        # gradients of a short clip in full precision, what a user compares a training run against
        _case("check_fp32", "train", "fp32", 1, 12, 24, 14, 4, 4),
        # the training step of the 310M model: 16 frames of 384 x 224, four clips a GPU
        _case("train", "train", "bf16", 4, 16, 24, 14, 16, 16),
        # long clips with larger frames: the largest call
        _case("train_long", "train", "bf16", 2, 16, 24, 24, 64, 64),
        # another aspect ratio and model size: frames, rows and heads that fit no tile
        _case("train_ragged", "train", "bf16", 1, 12, 19, 13, 11, 11),
        # teacher-forced evaluation of the same clips: forward alone
        _case("forward", "forward", "bf16", 4, 16, 24, 14, 16, 16),
        # interactive generation, one frame at a time over the 32-frame context
        _case("decode", "rope", "bf16", 1, 16, 24, 14, 33, 1, 40),
        # speculative generation, two frames a call, the context full: the window slides by two frames first
        _case("spec2_window", "rope", "bf16", 1, 16, 24, 14, 34, 2, 36, 2),
        # speculative generation, four frames a call, keys rotated by the caller
        _case("spec4", "step", "bf16", 1, 16, 24, 14, 36, 4, 40),
        # the start of a generation with the 130M model on an odd grid: few frames, short calls
        _case("decode_ragged", "rope", "bf16", 1, 12, 17, 11, 7, 1, 34),
        # serving eight sequences with a long context and larger frames
        _case("batch_decode", "step", "bf16", 8, 16, 24, 24, 64, 1, 64),
        # four speculative frames over the 8-bit cache
        _case("spec4_fp8", "rope8", "bf16", 1, 16, 24, 14, 36, 4, 40),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One case of the ranges the listed ones stand for: any grid up to 24 x 24, the models' head counts and others, up to
    64 frames of keys, up to eight new frames."""
    limit = max(work(c)["flops"] for c in listed())
    while True:
        kind = rng.choice(["forward", "train", "train", "step", "rope", "rope", "rope8"])
        dtype = rng.choice(["bf16", "bf16", "bf16", "fp32"]) if kind in ("forward", "train") else "bf16"
        H = rng.choice([12, 16, 24, rng.randint(1, 24)])
        gh, gw = _log_int(rng, 4, 24), _log_int(rng, 4, 24)
        if dtype == "fp32":  # full precision is for checks: short clips; the general path takes any head width
            D = rng.choice([64, 64, 32, 128])
            kv = n = _log_int(rng, 1, 8)
            c = _case("", kind, dtype, rng.randint(1, 2), H, gh, gw, kv, n, D=D)
        elif kind in ("forward", "train"):
            kv = _log_int(rng, 2, 64)
            c = _case("", kind, dtype, _log_int(rng, 1, 8), H, gh, gw, kv, kv)
        else:
            n = rng.choice([1, 1, 2, 3, 4, 8])
            past = _log_int(rng, 2, 63)
            drop = n if kind != "step" and rng.random() < 0.4 else 0
            c = _case("", kind, dtype, _log_int(rng, 1, 8), H, gh, gw, past + n, n, past + n + drop + rng.randint(0, 4), drop)
        if work(c)["flops"] <= limit:
            del c["name"]
            return c


def _pairs(c):
    past = c["kv"] - c["n"]
    return c["T"] ** 2 * (c["n"] * past + c["n"] * (c["n"] + 1) // 2) * c["B"] * c["H"]


def work(c):
    """Multiply-adds of the visible (query, key) pairs, two operations each: two products forward, five backward.  Bytes: every
    tensor the caller hands in or gets, once."""
    es = 4 if c["dtype"] == "fp32" else 2
    frame = c["B"] * c["H"] * c["T"] * c["D"]  # elements of one frame of one tensor
    new, past = c["n"] * frame, (c["kv"] - c["n"]) * frame
    pairs = _pairs(c)
    if c["kind"] == "train":  # q, k, v, dout in; out, log-sum-exp, dq, dk, dv out
        return {"bytes": 8 * new * es + 4 * new // c["D"], "flops": 14 * c["D"] * pairs}
    flops = 4 * c["D"] * pairs
    if c["kind"] == "forward":
        return {"bytes": 4 * new * es, "flops": flops}
    # the new frames' q, k, v in; out and the cache rows of the new frames out; the earlier frames of the cache in
    ce = 1 if c["kind"] == "rope8" else es
    b = 4 * new * es + 2 * new * ce + 2 * past * ce
    if c["kind"] != "step":
        b += new * es                # the rotated queries
    if c["drop"]:
        b += 2 * past * ce           # the kept frames written to their new place
    return {"bytes": b, "flops": flops}


def tolerance(c):
    # Measured against the same sequence of calls in float64 (relative 2-norm): bf16 outputs 2.3e-3 to 3.4e-3 (queries, P and
    # the key-split partials rounded to bf16 once each), gradients 2.2e-3 to 2.5e-3; float32 outputs and gradients 5e-8 to
    # 9e-7.  8-bit codes are decided in float32 from a rotated key rounded to bf16: a rotation summed otherwise may move
    # a rounding, hence a few codes.
    if c["dtype"] == "fp32":
        return {"rel": 4e-6}
    if c["kind"] == "rope8":
        return {"rel": 1e-2, "differ": 1e-4}
    return {"rel": 1e-2}


def prepare(c, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    B, H, D, T = c["B"], c["H"], c["D"], c["T"]

    def randn(frames):  # projected activations: zero mean, unit variance
        return torch.randn((B, H, frames * T, D), generator=gen, device="cuda", dtype=torch.float32).to(dt)

    s = {"case": c, "attn": nb.Attention(c["dtype"], torch.cuda.current_device())}
    s["q"] = randn(c["n"])
    if c["kind"] in ("forward", "train"):
        s["k"], s["v"] = randn(c["kv"]), randn(c["kv"])
        if c["kind"] == "train":
            s["dout"] = randn(c["n"])
        return s
    s["k_new"], s["v_new"] = randn(c["n"]), randn(c["n"])
    before = c["kv"] - c["n"] + c["drop"]  # frames in the cache when the step begins
    if c["kind"] == "rope8":
        s["k_scale"] = torch.full((B, H), FP8_SCALE, device="cuda")
        s["v_scale"] = torch.full((B, H), FP8_SCALE, device="cuda")
        nbytes = nb.nfd_fp8_cache_bytes(B, H, c["F"], T, D)
        s["kc"] = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        s["vc"] = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
        nb.nfd_kvcache_append_fp8(s["attn"].h, s["kc"], s["vc"], s["k_scale"], s["v_scale"], randn(before), randn(before),
                                  B, H, c["F"], T, D, 0, before)
    else:
        s["kc"] = torch.zeros((B, H, c["F"] * T, D), dtype=dt, device="cuda")
        s["vc"] = torch.zeros((B, H, c["F"] * T, D), dtype=dt, device="cuda")
        s["kc"][:, :, : before * T] = randn(before)
        s["vc"][:, :, : before * T] = randn(before)
    if c["kind"] == "step" or c["kind"] == "rope8":
        s["out"] = torch.empty_like(s["q"])
    if c["kind"] == "rope8":
        s["q_rot"] = torch.empty_like(s["q"])
    return s


def run(s):
    c, attn = s["case"], s["attn"]
    B, H, D, T, F, kv, n = c["B"], c["H"], c["D"], c["T"], c["F"], c["kv"], c["n"]
    kind = c["kind"]
    if kind == "forward":
        return attn.forward(s["q"], s["k"], s["v"], T)
    if kind == "train":
        out, lse = attn.forward_lse(s["q"], s["k"], s["v"], T)
        dq, dk, dv = attn.backward(s["q"], s["k"], s["v"], out, s["dout"], lse, T)
        return out, lse, dq, dk, dv
    kc, vc = s["kc"], s["vc"]
    if kind == "step":
        nb.nfd_kvcache_append_attn_fwd(attn.h, s["q"], kc, vc, s["k_new"], s["v_new"], s["out"], B, H, F, T, D, kv, n)
        return s["out"], kc, vc
    past = kv - n
    if kind == "rope":
        if c["drop"]:
            nb.nfd_kvcache_shift(attn.h, kc, vc, B, H, F, T, D, past + c["drop"], c["drop"])
        q_rot = attn.rope_append(s["q"], kc, vc, s["k_new"], s["v_new"], T, past, (c["gh"], c["gw"]), SECTIONS)
        return attn.forward(q_rot, kc, vc, T, kv_frames=kv, q_frames=n), q_rot, kc, vc
    if c["drop"]:
        nb.nfd_kvcache_shift_fp8(attn.h, kc, vc, B, H, F, T, D, past + c["drop"], c["drop"])
    nb.nfd_rope_kvcache_append_fp8(attn.h, s["q"], s["q_rot"], kc, vc, s["k_scale"], s["v_scale"], s["k_new"], s["v_new"], B, H,
                                   F, T, D, past, n, 0, c["gh"], c["gw"], *SECTIONS)
    nb.nfd_block_causal_attn_fwd_fp8kv(attn.h, s["q_rot"], kc, vc, s["k_scale"], s["v_scale"], s["out"], B, H, F, T, D, kv, n)
    return s["out"], s["q_rot"], kc, vc
