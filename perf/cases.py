"""The calls whose speed on one MI355X is measured, and how each is prepared, made and checked.

A case is one call (or, for the whole layer, one chain of calls) that an integer
Conformer encoder makes through the package's public classes: the relative-position
attention block alone and inside its residual module, the feed-forward module, the
convolution module, the LayerNorm, and the five of them chained as one encoder layer.
Sizes are those of the repository's own workloads (frames of 80 ms: T = 125 is 10 s of
audio, 375 is 30 s, 2500 is 200 s; d_model 256 and 1024, d_k 64 and 128, d_ff = 4 d)
and the ranges between and around them up to the block's limit of 8000 frames.

The path is integer only, so every output is a whole number that has one correct value.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_30846_amd import ipk
from workloads import make_block, make_conv, make_ffn, make_residual
from workloads.generate import ConfigShape

KINDS = ("block", "mhsa", "ffn", "conv", "layernorm", "layer")
MOST_FLOPS = 4.0e11  # the largest listed case's, which no drawn case exceeds


def listed():
    return [
        # the smallest block of the workloads: one 5 s command, nothing but latency
        {"name": "block_tiny", "kind": "block", "B": 1, "T": 64, "d": 256, "H": 4, "low": 64, "regime": "calibrated"},
        # one 10 s utterance, the interactive request
        {"name": "block_10s", "kind": "block", "B": 1, "T": 125, "d": 1024, "H": 8, "low": 125, "regime": "calibrated"},
        # sixteen utterances of 16 to 30 s padded to the longest, the batched request
        {"name": "block_batch", "kind": "block", "B": 16, "T": 375, "d": 1024, "H": 8, "low": 200,
         "regime": "calibrated"},
        # 200 s of audio in one piece, the benchmark's shape
        {"name": "block_longform", "kind": "block", "B": 1, "T": 2500, "d": 1024, "H": 8, "low": 2500,
         "regime": "calibrated"},
        # eight minutes in one piece, past what the wider query blocks hold on chip
        {"name": "block_8min", "kind": "block", "B": 1, "T": 6000, "d": 1024, "H": 8, "low": 6000,
         "regime": "calibrated"},
        # the attention module of an encoder layer of the stack workload, positions projected once at start-up
        {"name": "mhsa_stack", "kind": "mhsa", "B": 8, "T": 500, "d": 1024, "H": 8, "low": 500, "kept": True,
         "regime": "calibrated"},
        # the feed-forward module on one 10 s utterance, on a stack layer's rows, and on a full server batch
        {"name": "ffn_10s", "kind": "ffn", "rows": 125, "d": 1024, "d_ff": 4096},
        {"name": "ffn_stack", "kind": "ffn", "rows": 4000, "d": 1024, "d_ff": 4096},
        {"name": "ffn_server", "kind": "ffn", "rows": 23000, "d": 1024, "d_ff": 4096},
        # the convolution module on the batched request
        {"name": "conv_batch", "kind": "conv", "B": 16, "T": 375, "d": 1024, "low": 200},
        # the encoder's final LayerNorm over the batched request
        {"name": "layernorm_batch", "kind": "layernorm", "rows": 6000, "d": 1024},
        # a whole encoder layer (feed-forward, attention, convolution, feed-forward, LayerNorm) on 200 s of audio
        {"name": "layer_longform", "kind": "layer", "B": 1, "T": 2500, "d": 1024, "H": 8, "low": 2500},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        case = _draw(rng)
        if work(case)["flops"] <= MOST_FLOPS:
            return case


def _draw(rng):
    kind = rng.choices(KINDS, weights=(6, 3, 4, 4, 1, 2))[0]
    d = rng.choice((256, 512, 1024, 1024, 1024))
    if kind == "layernorm":
        return {"kind": kind, "rows": _log_int(rng, 400, 40000), "d": d}
    if kind == "ffn":
        return {"kind": kind, "rows": _log_int(rng, 16, 23000), "d": d, "d_ff": 4 * d}
    B = _log_int(rng, 1, 32)
    T = _log_int(rng, 40, 1600) if B > 1 else _log_int(rng, 40, 8000)
    low = T if rng.random() < 0.4 else max(1, int(T * rng.uniform(0.4, 1.0)))
    case = {"kind": kind, "B": B, "T": T, "d": d, "low": low}
    if kind == "conv":
        return case
    case["H"] = d // (64 if rng.random() < 0.25 else 128)
    if kind == "block":
        # (over many keys the literal regime's saturated scores leave every softmax code zero)
        case["regime"] = rng.choice(("calibrated", "literal")) if T <= 400 else "calibrated"
    if kind == "mhsa":
        case["regime"] = "calibrated"
        case["kept"] = rng.random() < 0.5
    return case


def _block(case, rng):
    lengths = rng.integers(case["low"], case["T"] + 1, size=case["B"])
    lengths[int(rng.integers(case["B"]))] = case["T"]  # padded to the longest
    shape = ConfigShape("case", B=case["B"], T=case["T"], d_model=case["d"], n_heads=case["H"])
    return make_block(shape, case["T"], rng, case.get("regime", "calibrated"), lengths=lengths)


def _rows(rng, rows, d):
    return np.clip(np.rint(rng.normal(0.0, 32.0, size=(rows, d))), -127, 127).astype(np.int8)


S_Z = 1.0 / 32.0  # grid of unit-variance activations with the standard deviation above


def _host(case, seed):
    """The integer parameters and inputs of a case, as the offline tools hand them over."""
    rng = np.random.default_rng(seed)
    kind, d = case["kind"], case["d"]
    h = {}
    if kind in ("block", "mhsa", "layer"):
        h["blk"] = _block(case, rng)
        h["x"], h["lengths"], h["pos"] = h["blk"].x, h["blk"].lengths, h["blk"].pos_table
    elif kind == "conv":
        h["x"] = _rows(rng, case["B"] * case["T"], d).reshape(case["B"], case["T"], d)
        h["lengths"] = rng.integers(case["low"], case["T"] + 1, size=case["B"]).astype(np.int32)
    else:
        h["x"] = _rows(rng, case["rows"], d)
    s = int(rng.integers(1 << 31))
    if kind in ("mhsa", "layer"):
        h["res"] = make_residual(h["blk"], "calibrated", seed=s)
    if kind in ("ffn", "layer"):
        h["ffn"] = make_ffn(d, "calibrated", seed=s + 1, S_z=S_Z, d_ff=case.get("d_ff", 4 * d))
    if kind in ("conv", "layer"):
        h["conv"] = make_conv(d, "calibrated", seed=s + 2, S_z=S_Z)
    if kind == "layer":
        h["ffn2"] = make_ffn(d, "calibrated", seed=s + 3, S_z=S_Z)
    if kind in ("layernorm", "layer"):
        h["ln"] = make_ffn(d, "calibrated", seed=s + 4, S_z=S_Z, d_ff=64)  # its LayerNorm constants alone
    return h


def prepare(case, seed):
    h = _host(case, seed)
    kind = case["kind"]
    st = {"kind": kind, "x": torch.from_numpy(h["x"]).cuda(), "lengths": h.get("lengths"), "pos": None}
    if kind in ("block", "mhsa", "layer"):
        st["attn"] = ipk.RelPosAttn.from_block(h["blk"])
        st["pos"] = torch.from_numpy(h["pos"]).cuda()
        if kind != "block":
            st["attn"].set_residual_from(h["res"])
        if case.get("kept"):
            st["attn"].cache_positions(st["pos"])
            st["pos"] = None
    rows = h["x"].size // case["d"]
    if kind in ("ffn", "layer"):
        st["ffn"] = ipk.FeedForward(h["ffn"], max_rows=rows)
    if kind in ("conv", "layer"):
        st["conv"] = ipk.ConvModule(h["conv"], max_batch=case["B"], max_T=case["T"])
    if kind == "layer":
        st["ffn2"] = ipk.FeedForward(h["ffn2"], max_rows=rows)
    if kind in ("layernorm", "layer"):
        st["ln"] = ipk.LayerNorm(case["d"], h["ln"])
    return st


def run(st):
    kind, x = st["kind"], st["x"]
    if kind == "block":
        return st["attn"](x, st["pos"], lengths=st["lengths"])
    if kind == "mhsa":
        return st["attn"].residual(x, st["pos"], lengths=st["lengths"])
    if kind == "ffn":
        return st["ffn"](x)
    if kind == "conv":
        return st["conv"](x, lengths=st["lengths"])
    if kind == "layernorm":
        return st["ln"](x)
    z = st["ffn"](x)
    z = st["attn"].residual(z, st["pos"], lengths=st["lengths"])
    z = st["conv"](z, lengths=st["lengths"])
    z = st["ffn2"](z)
    return z, st["ln"](z)


def work(case):
    """Operations are 2 x the multiply-accumulates.  Lengths are drawn, so padded frames
    count by the mean length; the parameters count once."""
    kind, d = case["kind"], case["d"]
    if kind == "layernorm":
        return {"bytes": 2.0 * case["rows"] * d + 12 * d, "flops": 0.0}
    if kind == "ffn":
        rows, f = case["rows"], case["d_ff"]
        return {"bytes": 2.0 * rows * d + 2.0 * d * f, "flops": 4.0 * rows * d * f}
    B, T, low = case["B"], case["T"], case["low"]
    padded = 2.0 * B * T * d
    mean = (low + T) / 2.0
    square = (low * low + low * T + T * T) / 3.0  # mean of L^2 over L in [low, T]
    conv = {"bytes": padded + 3.0 * d * d + 9 * d, "flops": 2.0 * B * mean * d * (3 * d + 9)}
    if kind == "conv":
        return conv
    projections = 4.0 * B * mean + (0 if case.get("kept") else 2 * T - 1)
    attn = {"bytes": padded + 5.0 * d * d + (2.0 * T - 1) * d,
            "flops": 2.0 * (projections * d * d + 3.0 * d * B * square)}
    if kind != "layer":
        return attn
    rows = B * T
    return {"bytes": attn["bytes"] + conv["bytes"] + 3 * padded + 16.0 * d * d,
            "flops": attn["flops"] + conv["flops"] + 2 * 16.0 * rows * d * d}


def tolerance(case):
    return "exact"  # integers from end to end: one correct value each


# ---------------------------------------------------------------------------------
# The same integers in plain torch: 64-bit integers, the matrix products in float64 (every
# partial sum is a whole number far below 2^53).


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def _rs(a, m, n, lim=127):
    return (((a * m) + (1 << (n - 1))) >> n).clamp(-lim, lim)


def _mm(a, b_t):
    return (a.double() @ b_t.double().T.contiguous()).to(torch.int64)


def _linear(x, w, mult, shift):
    return _rs(_mm(x, _dev(w)), _dev(mult).to(torch.int64), int(shift))


def _isqrt(v):
    r = torch.floor(torch.sqrt(v.double())).to(torch.int64)
    r = torch.where(r * r > v, r - 1, r)
    return torch.where((r + 1) * (r + 1) <= v, r + 1, r)


def _layernorm(z, p):
    d = z.shape[-1]
    mu = torch.div(2 * z.sum(-1, keepdim=True) + d, 2 * d, rounding_mode="floor")
    sigma = _isqrt(((z - mu) ** 2).sum(-1, keepdim=True)).clamp(min=1)
    u = ((z - mu) * torch.div(1 << 31, sigma, rounding_mode="floor")) >> 1
    n = int(p.ln_shift)
    return ((u * _dev(p.ln_mult).to(torch.int64) + _dev(p.ln_bias) + (1 << (n - 1))) >> n).clamp(-127, 127)


def _residual(z, y, p):
    return _rs(int(p.m_z) * z + int(p.m_y) * y, 1, int(p.shift_r))


def _poly(q, q_c, q_1):
    return (q.abs().clamp(max=int(q_c)) - int(q_c)) ** 2 + int(q_1)


def _swish(q, p):
    return _rs(-(q.abs() * _poly(q, p.sw_qc, p.sw_q1) + q * int(p.sw_q1)), int(p.m_sw), int(p.shift_sw))


def _ffn(z, p):
    h = _linear(_layernorm(z, p), p.w1, p.mult1, p.shift1)
    return _residual(z, _linear(_swish(h, p), p.w2, p.mult2, p.shift2), p)


def _conv(z, p, lengths):
    B, T, d = z.shape
    valid = (torch.arange(T, device=z.device)[None, :] < _dev(lengths)[:, None])[..., None]
    u = _linear(_layernorm(z, p).reshape(-1, d), p.w_pw1, p.mult_pw1, p.shift_pw1).reshape(B, T, 2 * d)
    a, b = u[..., :d], u[..., d:]
    gate = -(int(p.glu_q1) + torch.sign(b) * _poly(b, p.glu_qc, p.glu_q1))
    g = torch.where(valid, _rs(a * gate, int(p.m_glu), int(p.shift_glu)), 0)
    g = torch.nn.functional.pad(g, (0, 0, 4, 4))
    w = _dev(p.w_dw).to(torch.int64)
    acc = _dev(p.bias_dw).to(torch.int64) + sum(g[:, k:k + T] * w[:, k] for k in range(9))
    v = _rs(acc, _dev(p.mult_dw).to(torch.int64), int(p.shift_dw), 32767)
    o = torch.where(valid, _swish(v, p), 0)
    return _residual(z, _linear(o.reshape(-1, d), p.w_pw2, p.mult_pw2, p.shift_pw2).reshape(B, T, d), p)


def _attention(x, blk):
    B, T, d = x.shape
    H, c = blk.shape.n_heads, blk.consts
    dk = d // H
    q, k, v = (_linear(x.reshape(-1, d), getattr(blk, "w_" + n), c["mult_" + n], c["shift_" + n]).reshape(B, T, H, dk)
               for n in "qkv")
    p = _linear(_dev(blk.pos_table).to(torch.int64), blk.w_pos, c["mult_pos"], c["shift_pos"]).reshape(-1, H, dk)
    bu, bv = _dev(blk.pos_bias_u).to(torch.int64), _dev(blk.pos_bias_v).to(torch.int64)
    ctx = torch.zeros((B, T, H, dk), dtype=torch.int64, device=x.device)
    at = torch.arange(T, device=x.device)
    for b in range(B):
        L = int(blk.lengths[b])
        rel = at[None, :L] - at[:L, None] + T - 1
        for h in range(H):
            cont = _mm(q[b, :L, h] + bu[h], k[b, :L, h])
            pos = torch.gather(_mm(q[b, :L, h] + bv[h], p[:, h]), 1, rel)
            s = _rs(c["m_c"] * cont + c["m_p"] * pos, 1, c["shift_s"])
            dist = s.amax(1, keepdim=True) - s
            z = torch.div(dist, c["q_ln2"], rounding_mode="floor")
            e = ((z * c["q_ln2"] - dist + c["q_b"]) ** 2 + c["q_c"]) >> z.clamp(max=62)
            f = torch.div(1 << 32, e.sum(1, keepdim=True), rounding_mode="floor")
            a = ((e * f) >> 24).clamp(max=255)
            ctx[b, :L, h] = _rs(_mm(a, v[b, :L, h].T), c["m_o"], c["shift_o"])
    y = _linear(ctx.reshape(-1, d), blk.w_out, c["mult_out"], c["shift_out"]).reshape(B, T, d)
    return torch.where((at[None, :] < _dev(blk.lengths)[:, None])[..., None], y, 0)


def _mhsa(z, blk, res):
    return _residual(z, _attention(_layernorm(z, res), blk), res)


def exact(case, seed):
    h = _host(case, seed)
    kind, z = case["kind"], _dev(h["x"]).to(torch.int64)
    if kind == "block":
        return _attention(z, h["blk"])
    if kind == "mhsa":
        return _mhsa(z, h["blk"], h["res"])
    if kind == "ffn":
        return _ffn(z, h["ffn"])
    if kind == "conv":
        return _conv(z, h["conv"], h["lengths"])
    if kind == "layernorm":
        return _layernorm(z, h["ln"])
    z = _mhsa(_ffn(z, h["ffn"]), h["blk"], h["res"])
    z = _ffn(_conv(z, h["conv"], h["lengths"]), h["ffn2"])
    return z, _layernorm(z, h["ln"])
