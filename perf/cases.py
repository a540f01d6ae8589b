"""The workloads that the library's speed is measured on.

Every case is one call that a detector running on this library makes: a whole
encoder, one encoder block, one decoder layer, or one operator through its own
entry point.  All tensors are integers and every result is exact, so two
correct implementations agree in every value.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  weights, inputs, output and workspace on the GPU
  run(state)           one pass
  work(case)           bytes and operations the pass cannot do without
  tolerance(case)      "exact"
  exact(case, seed)    the result in 64-bit integers, by plain torch

Inputs: activations are rounded normal values (sigma 42, clipped to the int8
range, as calibrated activations are), weights and requantization constants
come from the package's own generators with the calibration that keeps most
outputs inside int8 ("wide").  Shiftmax scales are drawn in [8, 16]: int8 score
rows of hundreds of keys then have some keys that stand out, as attention has,
where a flatter exponential would round every 8-bit weight to zero.
"""
import math

import numpy as np
import torch

from paper_2607_24981_amd import ilw, synth

DEV = "cuda" if torch.cuda.is_available() else "cpu"


# ---------------------------------------------------------------------- cases
def _block(batch, gh, gw, wh, ww, dim, mlp=0):
    return {"kind": "block", "batch": batch, "gh": gh, "gw": gw, "wh": wh, "ww": ww, "dim": dim,
            "mlp": mlp or 4 * dim}


def _encoder(batch, gh, gw, wh, ww, dim, blocks):
    return {"kind": "encoder", "batch": batch, "gh": gh, "gw": gw, "wh": wh, "ww": ww, "dim": dim,
            "mlp": 4 * dim, "blocks": blocks}


def _attention(batch, gh, gw, wh, ww, heads, head_dim, s_d=-1):
    return {"kind": "attention", "batch": batch, "gh": gh, "gw": gw, "wh": wh, "ww": ww,
            "heads": heads, "head_dim": head_dim, "s_d": s_d}


def _decoder(batch, queries, dim, heads, side, mode, boxes):
    return {"kind": "decoder", "batch": batch, "queries": queries, "dim": dim, "heads": heads,
            "side": side, "mode": mode, "boxes": boxes}


def _deform(batch, queries, heads, head_dim, side, points, mode, boxes):
    return {"kind": "deform", "batch": batch, "queries": queries, "heads": heads,
            "head_dim": head_dim, "side": side, "points": points, "mode": mode, "boxes": boxes}


def _split(batch, tokens, branches, channels, out, per_channel):
    return {"kind": "split", "batch": batch, "tokens": tokens, "branches": branches,
            "channels": channels, "out": out, "per_channel": per_channel}


def _patch(batch, height, width, dim):
    return {"kind": "patch", "batch": batch, "height": height, "width": width, "dim": dim}


def _shiftmax(rows, cols, s_d=-1):
    return {"kind": "shiftmax", "rows": rows, "cols": cols, "s_d": s_d}


def _linear(m, n, k, bias=True):
    return {"kind": "linear", "m": m, "n": n, "k": k, "bias": bias}


def listed():
    cases = [
        # one block of the tiny encoder on a 256x256 image: the smallest call,
        # a handful of short launches
        ("block_t256_d192_b1", _block(1, 16, 16, 0, 0, 192)),
        # the tiny encoder on one 640x640 frame, the latency case of a camera
        # stream: 6 blocks, 20x20 windows and global attention in turn
        ("encoder_t1600_d192_b1", _encoder(1, 40, 40, 20, 20, 192, 6)),
        # the medium encoder on a batch of 8 frames: the largest call
        ("encoder_t1600_d384_b8", _encoder(8, 40, 40, 20, 20, 384, 10)),
        # one window block of the tiny encoder at batch 32: throughput serving
        ("block_t1600_d192_b32", _block(32, 40, 40, 20, 20, 192)),
        # one window block on a 432x608 frame, batch 3: 171-token windows that
        # fill no tile, 3078 tokens
        ("block_t1026_d384_b3", _block(3, 27, 38, 9, 19, 384)),
        # global attention of the medium encoder by itself, 4 frames, from
        # token-major Q | K | V with one calibrated denominator shift
        ("attention_t1600_h6_b4", _attention(4, 40, 40, 0, 0, 6, 64, 3)),
        # a decoder layer: 300 queries over three levels, 8 frames, nearest
        # sampling
        ("decoder_q300_d256_b8", _decoder(8, 300, 256, 8, 20, 0, False)),
        # the sampler by itself with reference boxes and bilinear weights
        ("deform_q300_h8_b8_boxes", _deform(8, 300, 8, 32, 20, 4, 1, True)),
        # the projector's split convolution over three feature maps, batch 32
        ("split_t1600_c3x192_n256_b32", _split(32, 1600, 3, 192, 256, True)),
        # patch embedding of 8 frames
        ("patch_640x640_d384_b8", _patch(8, 640, 640, 384)),
        # the score rows of the decoder's self-attention (8 frames, 8 heads,
        # 300 queries): rows that are no whole number of 16-byte chunks
        ("shiftmax_r19200_c300", _shiftmax(19200, 300)),
        # the class head over the decoder's queries (8 x 300), 91 classes
        # padded to 96
        ("linear_m2400_n96_k256", _linear(2400, 96, 256)),
    ]
    return [dict(c, name=n) for n, c in cases]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _grid(rng, most):
    """A token grid and a window that tiles it (0, 0: global attention)."""
    gh, gw = rng.randint(7, 45), rng.randint(7, 45)
    while gh * gw > most:
        gh, gw = max(7, gh - 3), max(7, gw - 3)
    if rng.random() < 0.4:
        return gh, gw, 0, 0
    wh = rng.choice([d for d in range(1, gh + 1) if gh % d == 0 and (d >= 5 or d == gh)])
    ww = rng.choice([d for d in range(1, gw + 1) if gw % d == 0 and (d >= 5 or d == gw)])
    return gh, gw, wh, ww


def draw(rng):
    kind = rng.choice(["block", "block", "encoder", "encoder", "attention", "decoder", "deform",
                       "split", "patch", "shiftmax", "linear"])
    if kind == "block":
        gh, gw, wh, ww = _grid(rng, 2025)
        dim = rng.choice([128, 192, 192, 256, 384, 384, 512, 768])
        most = max(1, 51200 * 192 // (gh * gw * dim))
        return _block(_log(rng, 1, most), gh, gw, wh, ww, dim)
    if kind == "encoder":
        gh, gw, wh, ww = rng.choice([(40, 40, 20, 20), (32, 32, 16, 16), (30, 40, 15, 20),
                                     (24, 40, 12, 20), (25, 42, 5, 14), (14, 14, 7, 7)])
        dim = rng.choice([192, 384])
        blocks = rng.randint(2, 10)
        most = 8 * 1600 * 10 * 384 // (gh * gw * blocks * dim)
        return _encoder(_log(rng, 1, min(most, 32)), gh, gw, wh, ww, dim, blocks)
    if kind == "attention":
        gh, gw, wh, ww = _grid(rng, 2025)
        head_dim = rng.choice([32, 64])
        heads = rng.randint(1, 12)
        return _attention(_log(rng, 1, max(1, 76800 // (gh * gw * heads))), gh, gw, wh, ww, heads,
                          head_dim, rng.choice([-1, -1, 3]))
    if kind == "decoder":
        dim, heads = rng.choice([(256, 8), (256, 4), (128, 4), (384, 12)])
        return _decoder(_log(rng, 1, 8), rng.choice([100, 300, 301, 500, 900]), dim, heads,
                        rng.choice([13, 16, 20]), rng.randint(0, 1), rng.random() < 0.5)
    if kind == "deform":
        heads, head_dim = rng.choice([(8, 32), (4, 64), (8, 16), (8, 48), (12, 32)])
        return _deform(_log(rng, 1, 16), _log(rng, 50, 900), heads, head_dim, rng.randint(7, 25),
                       rng.choice([2, 4, 4, 5]), rng.randint(0, 1), rng.random() < 0.5)
    if kind == "split":
        return _split(_log(rng, 1, 32), rng.choice([1600, 1024, 1050, 625]), rng.randint(2, 4),
                      rng.choice([192, 384]), rng.choice([128, 256, 384]), rng.random() < 0.5)
    if kind == "patch":
        return _patch(_log(rng, 1, 16), 16 * rng.randint(14, 40), 16 * rng.randint(14, 40),
                      rng.choice([192, 384, 768]))
    if kind == "shiftmax":
        cols = rng.choice([49, 100, 171, 256, 300, 400, 900, 1023, 1600])
        return _shiftmax(_log(rng, 300, 19200 * 1600 // cols), cols, rng.choice([-1, -1, 3]))
    return _linear(_log(rng, 1, 51200), 16 * _log(rng, 1, 96), 16 * _log(rng, 4, 96),
                   rng.random() < 0.8)


# --------------------------------------------------------------------- inputs
def _act(gen, *shape):
    """int8 activations, on the GPU."""
    x = torch.randn(*shape, generator=gen, device=DEV)
    return (x * 42.0).round_().clamp_(-127, 127).to(torch.int8)


def _ints(gen, lo, hi, *shape, dtype=torch.int32):
    return torch.randint(lo, hi + 1, shape, generator=gen, device=DEV).to(dtype)


def _levels(side):
    """Three levels, each half as wide as the one before, and their starts."""
    hw = np.array([[4 * side, 4 * side], [2 * side, 2 * side], [side, side]], np.int32)
    n = hw[:, 0] * hw[:, 1]
    return hw, np.concatenate([[0], np.cumsum(n)[:-1]]).astype(np.int32), int(n.sum())


def _deform_tensors(gen, B, Q, H, L, P, boxes):
    ref = _ints(gen, 0, 65535, B, Q, 2)
    if boxes:
        ref = torch.cat([ref, _ints(gen, 1 << 12, 1 << 15, B, Q, 2)], -1)
    offsets = (torch.randn(B, Q, H, L, P, 2, generator=gen, device=DEV) * 700).round()
    return ref.contiguous(), offsets.clamp(-2048, 2047).to(torch.int16), _act(gen, B, Q, H, L * P)


def _inputs(c, seed):
    """Host parameters and device tensors of a case, from the seed alone."""
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind = c["kind"]
    if kind in ("block", "encoder"):
        params = [synth.block_params(rng, c["dim"], c["dim"] // 64, 64, c["mlp"], "wide")
                  for _ in range(c.get("blocks", 1))]
        for p in params:
            p["smax_I0"] = int(rng.integers(8, 17))
        return params, {"x": _act(gen, c["batch"], c["gh"] * c["gw"], c["dim"])}
    if kind == "attention":
        D = c["heads"] * c["head_dim"]
        p = synth.block_params(rng, 64, 1, 64, 64, "wide", smax_s_d=c["s_d"])
        p["smax_I0"] = int(rng.integers(8, 17))
        p["score_shift"] = 37 + (c["head_dim"] == 64)  # normal Q and K: scores within int8
        return p, {"qkv": _act(gen, c["batch"], c["gh"] * c["gw"], 3 * D)}
    if kind == "decoder":
        hw, start, S = _levels(c["side"])
        p = synth.decoder_params(rng, c["dim"], c["heads"], 4 * c["dim"], 3, 4, mode=c["mode"])
        p["ref_dims"] = 4 if c["boxes"] else 2
        p["smax_I0"] = int(rng.integers(8, 17))
        B, Q = c["batch"], c["queries"]
        t = {"tgt": _act(gen, B, Q, c["dim"]), "memory": _act(gen, B, S, c["dim"])}
        t["ref"] = _deform_tensors(gen, B, Q, 1, 1, 1, c["boxes"])[0]
        return p, t
    if kind == "deform":
        hw, start, S = _levels(c["side"])
        p = {"I0": 16, "out_mult": int(rng.integers(1 << 29, 1 << 30)), "out_shift": 35}
        ref, off, lg = _deform_tensors(gen, c["batch"], c["queries"], c["heads"], 3, c["points"],
                                       c["boxes"])
        return p, {"value": _act(gen, c["batch"], S, c["heads"], c["head_dim"]), "ref": ref,
                   "offsets": off, "logits": lg}
    if kind == "split":
        wl = synth.SplitConvWorkload("", 1, 1, (c["channels"],) * c["branches"], c["out"])
        p = synth.split_conv_inputs(wl, int(rng.integers(1 << 31)), per_channel=c["per_channel"])
        M = c["batch"] * c["tokens"]
        return p, {"xs%d" % i: _act(gen, M, c["channels"]) for i in range(c["branches"])}
    if kind == "patch":
        p = synth.patch_embed_inputs(int(rng.integers(1 << 31)), 1, c["dim"], c["height"],
                                     c["width"])
        return p, {"img": _act(gen, c["batch"], 3, c["height"], c["width"])}
    if kind == "shiftmax":
        return {"I0": int(rng.integers(8, 17))}, {"x": _act(gen, c["rows"], c["cols"])}
    K, N = c["k"], c["n"]
    p = {"w": rng.integers(-127, 128, (N, K)).astype(np.int8),
         "b": rng.integers(-(1 << 15), 1 << 15, N).astype(np.int32) if c["bias"] else None,
         "mult": rng.integers(1 << 29, 1 << 30, N).astype(np.int32),
         "shift": rng.integers(39, 42, N).astype(np.int32)}
    return p, {"x": _act(gen, c["m"], K)}


def prepare(case, seed):
    """What a program keeps between calls (device weights, workspace, output
    buffer) and one call's inputs."""
    p, t = _inputs(case, seed)
    kind = case["kind"]
    st = {"case": case, "p": p, **t}
    dev = ilw.to_device

    def buffer(n):
        return torch.empty(max(n, 16), dtype=torch.int8, device=DEV)

    if kind == "block":
        st["block"] = ilw.DeviceBlock(p[0], DEV)
        st["ws"] = buffer(st["block"].workspace_bytes(case["batch"], case["gh"], case["gw"],
                                                      case["wh"], case["ww"]))
        st["y"] = torch.empty_like(t["x"])
    elif kind == "encoder":
        # window attention and global attention in turn, window first
        win = [(case["wh"], case["ww"]) if i % 2 == 0 else (0, 0) for i in range(case["blocks"])]
        st["enc"] = ilw.Encoder(p, win, case["gh"], case["gw"], DEV)
        st["ws"] = st["enc"].workspace(case["batch"])
        st["y"] = torch.empty_like(t["x"])
    elif kind == "attention":
        D = case["heads"] * case["head_dim"]
        st["ws"] = buffer(ilw.lib().ilw_attention_workspace_bytes(
            case["batch"], case["gh"], case["gw"], case["wh"], case["ww"], D, case["head_dim"]))
        st["y"] = torch.empty(case["batch"], case["gh"] * case["gw"], D, dtype=torch.int8,
                              device=DEV)
    elif kind == "decoder":
        st["dec"] = ilw.DeviceDecoder(p, DEV)
        st["hw"], st["start"], S = _levels(case["side"])
        st["ws"] = buffer(st["dec"].workspace_bytes(case["batch"], case["queries"], S))
        st["y"] = torch.empty_like(t["tgt"])
    elif kind == "deform":
        st["hw"], st["start"], _ = _levels(case["side"])
        st["y"] = torch.empty(case["batch"], case["queries"], case["heads"] * case["head_dim"],
                              dtype=torch.int8, device=DEV)
    elif kind == "split":
        st["xs"] = [t["xs%d" % i] for i in range(case["branches"])]
        for k in ("ws", "branch_mults", "branch_shifts"):
            st[k] = [dev(a, DEV) for a in p[k]]
        for k in ("bias", "out_mult", "out_shift"):
            st[k] = dev(p[k], DEV)
        st["y"] = torch.empty(case["batch"] * case["tokens"], case["out"], dtype=torch.int8,
                              device=DEV)
    elif kind == "patch":
        for k in ("w", "bias", "mult", "shift", "pos"):
            st[k] = dev(p[k], DEV)
        st["y"] = torch.empty(case["batch"], p["pos"].shape[0], case["dim"], dtype=torch.int8,
                              device=DEV)
    elif kind == "shiftmax":
        st["y"] = torch.empty_like(t["x"])
    else:
        st["w"], st["mult"], st["shift"] = (dev(p[k], DEV) for k in ("w", "mult", "shift"))
        st["b"] = None if p["b"] is None else dev(p["b"], DEV)
        st["y"] = torch.empty(case["m"], case["n"], dtype=torch.int8, device=DEV)
    return st


def run(st):
    c, kind, p = st["case"], st["case"]["kind"], st["p"]
    if kind == "block":
        return ilw.ilw_block_forward(st["block"], st["x"], c["gh"], c["gw"], c["wh"], c["ww"],
                                     y=st["y"], workspace=st["ws"])
    if kind == "encoder":
        return st["enc"].forward(st["x"], out=st["y"], workspace=st["ws"])
    if kind == "attention":
        return ilw.ilw_attention(st["qkv"], c["gh"], c["gw"], c["wh"], c["ww"], c["heads"], p,
                                 out=st["y"], workspace=st["ws"])
    if kind == "decoder":
        return ilw.ilw_decoder_layer(st["dec"], st["tgt"], st["memory"], st["ref"], st["hw"],
                                     st["start"], y=st["y"], workspace=st["ws"])
    if kind == "deform":
        call = ilw.ilw_deform_attn_boxes if c["boxes"] else ilw.ilw_deform_attn
        return call(st["value"], st["hw"], st["start"], st["ref"], st["offsets"], st["logits"],
                    p["I0"], p["out_mult"], p["out_shift"], mode=c["mode"], out=st["y"])
    if kind == "split":
        return ilw.ilw_split_conv(st["xs"], st["ws"], st["branch_mults"], st["branch_shifts"],
                                  st["bias"], st["out_mult"], st["out_shift"], y=st["y"])
    if kind == "patch":
        return ilw.ilw_patch_embed(st["img"], st["w"], st["bias"], st["mult"], st["shift"],
                                   st["pos"], p["pos_mult_a"], p["pos_mult_b"], p["pos_shift"],
                                   y=st["y"])
    if kind == "shiftmax":
        return ilw.ilw_shiftmax(st["x"], p["I0"], s_d=c["s_d"], y=st["y"])
    return ilw.ilw_linear(st["x"], st["w"], st["b"], st["mult"], st["shift"], y=st["y"])


# ----------------------------------------------------------------------- work
def work(case):
    """Inputs and weights read once, outputs written once; two operations per
    multiply-accumulate of the contractions."""
    c, kind = case, case["kind"]
    if kind in ("block", "encoder"):
        T, D, F, n = c["gh"] * c["gw"], c["dim"], c["mlp"], c.get("blocks", 1)
        weights = 4 * D * D + 2 * D * F + 12 * (6 * D + F + D)
        keys = [(c["wh"] * c["ww"] or T) if kind == "block" or i % 2 == 0 else T for i in range(n)]
        flops = sum(2 * T * (4 * D * D + 2 * D * F) + 4 * T * k * D for k in keys)
        return {"bytes": 2 * c["batch"] * T * D + n * weights, "flops": c["batch"] * flops}
    if kind == "attention":
        T, D = c["gh"] * c["gw"], c["heads"] * c["head_dim"]
        keys = c["wh"] * c["ww"] or T
        return {"bytes": 4 * c["batch"] * T * D, "flops": 4 * c["batch"] * T * keys * D}
    if kind == "decoder":
        B, Q, D, H = c["batch"], c["queries"], c["dim"], c["heads"]
        S = _levels(c["side"])[2]
        lin = D * (3 * D + D + 36 * H + D + 8 * D)
        byts = B * (2 * Q * D + S * D + Q * (16 if c["boxes"] else 8)) + lin + D * D
        return {"bytes": byts, "flops": 2 * B * (Q * lin + S * D * D + 2 * Q * Q * D)}
    if kind == "deform":
        n = c["batch"] * c["queries"] * c["heads"]
        LP, Dh = 3 * c["points"], c["head_dim"]
        # the whole value map, or less where the samples cannot touch all of it
        taps = n * LP * Dh * (4 if c["mode"] else 1)
        value = c["batch"] * _levels(c["side"])[2] * c["heads"] * Dh
        ref = c["batch"] * c["queries"] * (16 if c["boxes"] else 8)
        return {"bytes": min(value, taps) + ref + n * (LP * 5 + Dh), "flops": 2 * taps}
    if kind == "split":
        M, K, N = c["batch"] * c["tokens"], c["branches"] * c["channels"], c["out"]
        return {"bytes": M * K + K * N + M * N, "flops": 2 * M * N * K}
    if kind == "patch":
        T, D = c["height"] * c["width"] // 256, c["dim"]
        return {"bytes": c["batch"] * T * (768 + D) + 769 * D + T * D,
                "flops": 2 * c["batch"] * T * 768 * D}
    if kind == "shiftmax":
        return {"bytes": 2 * c["rows"] * c["cols"], "flops": 0}
    return {"bytes": c["m"] * (c["k"] + c["n"]) + c["k"] * c["n"],
            "flops": 2 * c["m"] * c["n"] * c["k"]}


def tolerance(case):
    """Integer arithmetic throughout: every correct result is the same."""
    return "exact"


# ------------------------------------------------------- the result in 64 bits
def _t(a):
    return torch.as_tensor(np.asarray(a), device=DEV).long()


def _sat(v):
    return v.clamp(-127, 127)


def _rq(acc, mult, shift):
    """Dyadic rescale, round half up, to int8: ((a m >> (s - 1)) + 1) >> 1
    rounds like (a m + 2^(s-1)) >> s without its overflow."""
    mult, shift = (v if torch.is_tensor(v) else _t(v) for v in (mult, shift))
    return _sat((((acc * mult) >> (shift - 1)) + 1) >> 1)


def _mm(a, b):
    """a [.., M, K] times b [.., N, K] transposed; the integers are exact in
    the doubles (below 2^53)."""
    return (a.double() @ b.double().transpose(-1, -2).contiguous()).long()


def _lin(x, p, stem):
    acc = _mm(x, _t(p["w_" + stem])) + _t(p["b_" + stem])
    return _rq(acc, p[stem + "_mult"], p[stem + "_shift"])


def _res(a, b, ma, mb, s):
    return _sat((a * ma + b * mb + (1 << (s - 1))) >> s)


def _exp(i, I0, k):
    """Integer exponential of i <= 0 at scale 1 / I0, times 2^k."""
    z = torch.clamp(i + (i >> 1) - (i >> 4), min=-k * I0)
    n = torch.div(-z, I0, rounding_mode="floor")
    return (((z + n * I0) >> 1) + I0) << (k - n)


def _softmax(x, I0, s_d=-1, k=16, k_out=8, m_p=4):
    """Constrained Shiftmax over the last axis."""
    table = _exp(-torch.arange(256, device=DEV), I0, k)
    e = table[x.amax(-1, keepdim=True) - x]
    s = e.sum(-1, keepdim=True)
    if s_d < 0:  # bit length of s - 1, plus the margin, past the 31 bits there are
        bits = torch.frexp((s - 1).double())[1].long()
        sd = (bits + m_p - 31).clamp(min=0)
    else:
        sd = torch.full_like(s, s_d)
    f = torch.div(2**31 - 1, (s >> sd).clamp(1, 2**31 - 1), rounding_mode="floor")
    return ((e * f) >> (32 - k_out + sd)).clamp(max=2**(k_out - 1) - 1)


def _gelu(x, p):
    I0, k, k_out = p["gelu_I0"], p["gelu_k_inter"], p["gelu_k_out"]
    v = torch.arange(-128, 128, device=DEV)
    z = v + (v >> 1) + (v >> 3) + (v >> 4)
    one, t = I0 << k, _exp(-z.abs(), I0, k)
    ratio = (torch.div(2**31 - 1, one + t, rounding_mode="floor") *
             torch.where(z >= 0, torch.full_like(t, one), t)) >> (32 - k_out)
    return _rq(v * ratio, p["gelu_mult"], p["gelu_shift"])[x + 128]


def _norm(x, p, stem):
    C = x.shape[-1]
    mu = torch.div(2 * x.sum(-1, keepdim=True) + C, 2 * C, rounding_mode="floor")
    d = x - mu
    V = (d * d).sum(-1, keepdim=True)
    k = torch.full_like(V, 1 << 16)
    for _ in range(p["ln_iters"]):
        k = (k + torch.div(V, k.clamp(min=1), rounding_mode="floor")) >> 1
    F = torch.where(V > 0, torch.div(2**31 - 1, k.clamp(min=1), rounding_mode="floor"),
                    torch.zeros_like(V))
    return _rq(((d * F) >> 1) + _t(p[stem + "_beta"]), p[stem + "_mult"], p[stem + "_shift"])


def _attend(qkv, p, gh, gw, wh, ww, H):
    """[T, 3D] of one image -> [T, D]."""
    wh, ww = wh or gh, ww or gw
    D = qkv.shape[-1] // 3
    tok = torch.arange(gh * gw, device=DEV).view(gh // wh, wh, gw // ww, ww)
    tok = tok.permute(0, 2, 1, 3).reshape(-1, wh * ww)
    q, k, v = qkv[tok].view(*tok.shape, 3, H, D // H).permute(2, 0, 3, 1, 4)  # [nW, H, Tw, d]
    out = torch.empty(gh * gw, D, dtype=torch.int64, device=DEV)
    for w in range(tok.shape[0]):
        s = _rq(_mm(q[w], k[w]), p["score_mult"], p["score_shift"])
        o = _mm(_softmax(s, p["smax_I0"], p["smax_s_d"]), v[w].transpose(-1, -2))
        o = _rq(o, p["pv_mult"], p["pv_shift"])
        out[tok[w]] = o.permute(1, 0, 2).reshape(-1, D)
    return out


def _block_exact(x, p, gh, gw, wh, ww):
    a = _attend(_lin(_norm(x, p, "ln1"), p, "qkv"), p, gh, gw, wh, ww, p["heads"])
    x1 = _res(_lin(a, p, "proj"), x, p["res1_mult_a"], p["res1_mult_b"], p["res1_shift"])
    g = _gelu(_lin(_norm(x1, p, "ln2"), p, "fc1"), p)
    return _res(_lin(g, p, "fc2"), x1, p["res2_mult_a"], p["res2_mult_b"], p["res2_shift"])


def _sample(value, hw, start, ref, off, lg, P, I0, mult, shift, mode, s_d=-1):
    """value [B, S, H, Dh], off [B, Q, H, L, P, 2] -> [B, Q, H * Dh]."""
    B, S, H, Dh = value.shape
    Q, L = off.shape[1], off.shape[3]
    wgt = _softmax(lg, I0, s_d).view(B, Q, H, L, P)
    acc = torch.zeros(B, Q, H, Dh, dtype=torch.int64, device=DEV)
    bi = torch.arange(B, device=DEV).view(B, 1, 1, 1)
    hi = torch.arange(H, device=DEV).view(1, 1, H, 1)
    r = ref.view(B, Q, 1, 1, -1)
    for l in range(L):
        h, w = int(hw[l][0]), int(hw[l][1])
        at = []
        for i, n in ((0, w), (1, h)):
            o = off[:, :, :, l, :, i]
            if ref.shape[-1] == 2:
                at.append(((r[..., i] * n) >> 8) + o)
            else:
                at.append(torch.div((r[..., i] * 512 * P + o * r[..., 2 + i]) * n, 131072 * P,
                                    rounding_mode="floor"))
        taps = []
        if mode == 0:
            taps.append((at[0] >> 8, at[1] >> 8, 1))
        else:
            X, Y = at[0] - 128, at[1] - 128
            fx, fy = X & 255, Y & 255
            for dy in (0, 1):
                for dx in (0, 1):
                    taps.append(((X >> 8) + dx, (Y >> 8) + dy,
                                 (fx if dx else 256 - fx) * (fy if dy else 256 - fy)))
        for ix, iy, t in taps:
            inside = (ix >= 0) & (ix < w) & (iy >= 0) & (iy < h)
            row = int(start[l]) + iy.clamp(0, h - 1) * w + ix.clamp(0, w - 1)
            tw = wgt[:, :, :, l] * t * inside
            acc += (value[bi, row, hi] * tw.unsqueeze(-1)).sum(3)
    return _rq(acc, mult, shift + (16 if mode else 0)).reshape(B, Q, H * Dh)


def _int8(v):
    return v.to(torch.int8)


def exact(case, seed):
    c, kind = case, case["kind"]
    p, t = _inputs(case, seed)
    if kind in ("block", "encoder"):
        out = []
        for x in t["x"]:
            x = x.long()
            for i, bp in enumerate(p):
                win = (c["wh"], c["ww"]) if i % 2 == 0 else (0, 0)
                x = _block_exact(x, bp, c["gh"], c["gw"], *win)
            out.append(_int8(x))
        return torch.stack(out)
    if kind == "attention":
        return torch.stack([_int8(_attend(x.long(), p, c["gh"], c["gw"], c["wh"], c["ww"],
                                          c["heads"])) for x in t["qkv"]])
    if kind == "decoder":
        hw, start, S = _levels(c["side"])
        B, Q, D, H = c["batch"], c["queries"], c["dim"], c["heads"]
        tgt, mem = t["tgt"].long(), t["memory"].long()
        a = torch.stack([_attend(_lin(x, p, "qkv"), p, 1, Q, 0, 0, H) for x in tgt])

        def add(a, b, i):
            return _norm(_res(a, b, p["res%d_mult_a" % i], p["res%d_mult_b" % i],
                              p["res%d_shift" % i]), p, "ln%d" % i)

        t1 = add(_lin(a, p, "o"), tgt, 1)
        v = _lin(mem, p, "val").view(B, S, H, D // H)
        off = 16 * _lin(t1, p, "off").view(B, Q, H, 3, 4, 2)
        s = _sample(v, hw, start, t["ref"].long(), off, _lin(t1, p, "attw").view(B, Q, H, 12), 4,
                    p["da_I0"], p["da_out_mult"], p["da_out_shift"], c["mode"], p["da_s_d"])
        t2 = add(_lin(s, p, "co"), t1, 2)
        return _int8(add(_lin(_gelu(_lin(t2, p, "fc1"), p), p, "fc2"), t2, 3))
    if kind == "deform":
        hw, start, _ = _levels(c["side"])
        return _int8(_sample(t["value"].long(), hw, start, t["ref"].long(), t["offsets"].long(),
                             t["logits"].long(), c["points"], p["I0"], p["out_mult"],
                             p["out_shift"], c["mode"]))
    if kind == "split":
        total = _t(p["bias"])
        for i in range(c["branches"]):
            m, s = _t(p["branch_mults"][i]), _t(p["branch_shifts"][i])
            acc = _mm(t["xs%d" % i].long(), _t(p["ws"][i]))
            total = total + ((acc * m + (1 << (s - 1))) >> s)
        return _int8(_rq(total, p["out_mult"], p["out_shift"]))
    if kind == "patch":
        B, gh, gw = c["batch"], c["height"] // 16, c["width"] // 16
        x = t["img"].long().view(B, 3, gh, 16, gw, 16).permute(0, 2, 4, 1, 3, 5)
        y = _mm(x.reshape(B, gh * gw, 768), _t(p["w"])) + _t(p["bias"])
        return _int8(_res(_rq(y, p["mult"], p["shift"]), _t(p["pos"]), p["pos_mult_a"],
                          p["pos_mult_b"], p["pos_shift"]))
    if kind == "shiftmax":
        return torch.cat([_int8(_softmax(x.long(), p["I0"], c["s_d"]))
                          for x in t["x"].split(1 + (1 << 25) // c["cols"])])
    y = _mm(t["x"].long(), _t(p["w"]))
    if p["b"] is not None:
        y = y + _t(p["b"])
    return _int8(_rq(y, p["mult"], p["shift"]))
