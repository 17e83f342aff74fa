"""Workloads of the stick-breaking attention library, through its Python entry points.

A case names one way a program uses the library and the sizes it uses it at:

    kind      entry points                                  what the program is
    decode    sb_attn_decode                                one generated token against a kv cache
    prefill   sb_attn_fwd / sb_attn_fwd_gqa (without m)     a prompt, or a document that is scored
    halt      sb_attn_fwd_halt                              the same, stopping once the stick is used up
    train     sb_attn_fwd_train + sb_attn_bwd, or the       one training step of the attention of a
              _gqa forms (grouped kv heads, remainder bias) layer: forward, then all gradients
    packed    sb_attn_varlen_fwd + sb_attn_varlen_bwd       the same on a padding-free packed batch
    f32       sb_attn_fwd_f32                               full-precision forward

    B, H, Hkv, T, d   batch, query heads, kv heads, rows (decode: valid rows of the cache), head size
    cap               decode: allocated rows of the cache per head
    bias              remainder bias: one embedding per head, and its gradient in training
    eps               halt: the share of the stick that may be left unassigned
    cut               packed: seed of the lengths (T is their sum, longest the longest of them)

Outputs and workspaces are left to the entry points, as in the README's example; what a program has
in hand beforehand (activations, upstream gradient, cache, offsets, embeddings) is prepare()'s.
"""
import math
import random

import torch

from paper_2410_17980_amd import binding as sb

HEAD_DIMS = (32, 64, 128)
MOST_FLOPS = 2.2e12          # forward at B1 H32 T16384 d128
MOST_CACHE = 1.1e9           # bytes of the kv cache at B8 Hkv16 T16384 d128


def _case(name, kind, B, H, Hkv, T, d, **more):
    return {"name": name, "kind": kind, "B": B, "H": H, "Hkv": Hkv, "T": T, "d": d, **more}


def listed():
    return [
        # the first tokens of a chat on a model with 12 query and 4 kv heads: one short launch after another
        _case("decode_short", "decode", 1, 12, 4, 333, 128, cap=4096, bias=False),
        # a serving batch far into its 16K context
        _case("decode_batch", "decode", 8, 16, 16, 16384, 128, cap=16384, bias=False),
        # one request at the far end of a 64K context, grouped kv heads and remainder bias
        _case("decode_64k", "decode", 1, 32, 8, 65000, 128, cap=65536, bias=True),
        # a short prompt
        _case("prefill_short", "prefill", 1, 16, 16, 100, 64, bias=False),
        # a 16K-token document on a model with head size 128: length generalisation
        _case("prefill_16k", "prefill", 1, 32, 32, 16384, 128, bias=False),
        # the same evaluation on the 1B model (24 heads of 64), batch 1, with early halt
        _case("halt_16k", "halt", 1, 24, 24, 16384, 64, eps=1e-9),
        # training steps: the 1B-like shape, the 350M-like shape, a small ragged batch, and a model with
        # grouped kv heads and remainder bias
        _case("train_1b", "train", 8, 16, 16, 4096, 128, bias=False),
        _case("train_350m", "train", 8, 16, 16, 2048, 64, bias=False),
        _case("train_small", "train", 2, 4, 4, 777, 32, bias=False),
        _case("train_grouped", "train", 4, 12, 4, 2048, 128, bias=True),
        # padding-free training on documents of very different lengths
        _case("packed_1b", "packed", 1, 24, 24, 16384, 64, bias=False, longest=4096, cut=1),
        # the full-precision forward that results are checked against
        _case("f32_check", "f32", 1, 1, 1, 256, 64),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi))))))


def draw(rng):
    while True:
        kind = rng.choice(("decode",) * 3 + ("prefill", "prefill", "halt") + ("train",) * 4 + ("packed", "f32"))
        d = rng.choice(HEAD_DIMS)
        group = rng.choice((1, 1, 2, 3, 4, 8))
        bias = rng.random() < 0.3
        if kind == "decode":
            Hkv = _log_int(rng, 1, 32)
            T = _log_int(rng, 64, 65536)
            c = {"kind": kind, "B": _log_int(rng, 1, 32), "H": Hkv * group, "Hkv": Hkv, "T": T, "d": d,
                 "cap": T + rng.randrange(0, 1 + T // 4), "bias": bias}
            ok = Hkv * group <= 64 and c["B"] * Hkv * c["cap"] * d * 4 <= MOST_CACHE
        elif kind == "prefill":
            Hkv = _log_int(rng, 1, 32)
            c = {"kind": kind, "B": _log_int(rng, 1, 16), "H": Hkv * group, "Hkv": Hkv,
                 "T": _log_int(rng, 64, 16384), "d": d, "bias": bias}
            ok = Hkv * group <= 32 and work(c)["flops"] <= MOST_FLOPS
        elif kind == "halt":
            H = _log_int(rng, 1, 32)
            c = {"kind": kind, "B": _log_int(rng, 1, 16), "H": H, "Hkv": H, "T": _log_int(rng, 256, 16384), "d": d,
                 "eps": rng.choice((1e-4, 1e-6, 1e-9))}
            ok = work(c)["flops"] <= MOST_FLOPS
        elif kind == "train":
            Hkv = _log_int(rng, 1, 24)
            c = {"kind": kind, "B": _log_int(rng, 1, 16), "H": Hkv * group, "Hkv": Hkv,
                 "T": _log_int(rng, 64, 8192), "d": d, "bias": bias}
            ok = Hkv * group <= 32 and work(c)["flops"] <= 0.87 * MOST_FLOPS
        elif kind == "packed":
            Hkv = _log_int(rng, 1, 24)
            longest = _log_int(rng, 128, 8192)
            c = {"kind": kind, "B": 1, "H": Hkv * group, "Hkv": Hkv, "T": longest * rng.randrange(2, 9) + rng.randrange(64),
                 "d": d, "bias": bias, "longest": longest, "cut": rng.randrange(1 << 20)}
            ok = Hkv * group <= 32 and c["T"] <= 32768 and work(c)["flops"] <= 0.87 * MOST_FLOPS
        else:
            H = _log_int(rng, 1, 8)
            c = {"kind": kind, "B": _log_int(rng, 1, 4), "H": H, "Hkv": H, "T": _log_int(rng, 64, 2048), "d": d}
            ok = True
        if ok:
            return c


def lengths(case):
    """Lengths of a packed batch's sequences: the longest one, and others spread over the logarithm."""
    rng = random.Random(case["cut"])
    got, left = [case["longest"]], case["T"] - case["longest"]
    while left > 0:
        got.append(min(left, _log_int(rng, min(32, case["longest"]), case["longest"])))
        left -= got[-1]
    rng.shuffle(got)
    return got


def _activations(gen, shape_q, shape_kv, heads_at, dtype):
    """q, k, v with N(0,1) entries, by kv head in turn: as they are (the stick is used up within tens of
    keys), with k * 3 (sharp, nearly saturated weights), and with logits around -6 (weights that
    reach over hundreds and thousands of keys)."""
    randn = lambda shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32)
    q, k, v = randn(shape_q), randn(shape_kv), randn(shape_kv).to(dtype)
    d, H, Hkv = shape_q[-1], shape_q[heads_at], shape_kv[heads_at]
    far = math.sqrt(6.0 * math.sqrt(d))
    for h in range(Hkv):
        one = k.select(heads_at, h)
        if h % 3 == 1:
            one.mul_(3.0)
        elif h % 3 == 2:
            one[..., d - 1] = -far
            q.narrow(heads_at, h * (H // Hkv), H // Hkv)[..., d - 1] = far
    return q.to(dtype), k.to(dtype), v


def prepare(case, seed):
    kind, B, H, Hkv, T, d = (case[n] for n in ("kind", "B", "H", "Hkv", "T", "d"))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    randn = lambda *shape: torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)
    s = {"case": dict(case)}
    if kind == "decode":
        s["q"], s["k"], s["v"] = _activations(gen, (B, H, d), (B, Hkv, case["cap"], d), 1, torch.bfloat16)
    elif kind == "packed":
        s["q"], s["k"], s["v"] = _activations(gen, (H, T, d), (Hkv, T, d), 0, torch.bfloat16)
        ends = [0]
        for n in lengths(case):
            ends.append(ends[-1] + n)
        s["cu"] = torch.tensor(ends, dtype=torch.int32, device="cuda")
        s["dout"] = randn(H, T, d)
    else:
        dtype = torch.float32 if kind == "f32" else torch.bfloat16
        s["q"], s["k"], s["v"] = _activations(gen, (B, H, T, d), (B, Hkv, T, d), 1, dtype)
        if kind == "train":
            s["dout"] = randn(B, H, T, d)
    s["r"] = randn(H, d) if case.get("bias") else None
    return s


def run(s):
    c, q, k, v, r = s["case"], s["q"], s["k"], s["v"], s["r"]
    kind = c["kind"]
    if kind == "decode":
        return sb.sb_attn_decode(q, k, v, T=c["T"], r=r)
    if kind == "halt":
        return sb.sb_attn_fwd_halt(q, k, v, c["eps"])
    if kind == "f32":
        return sb.sb_attn_fwd_f32(q, k, v)
    if kind == "packed":
        o, m = sb.sb_attn_varlen_fwd(q, k, v, s["cu"], c["longest"], r=r)
        return (o, m) + sb.sb_attn_varlen_bwd(q, k, v, m, s["dout"], s["cu"], c["longest"], r=r)
    plain = r is None and c["H"] == c["Hkv"]
    if kind == "prefill":
        return sb.sb_attn_fwd(q, k, v) if plain else sb.sb_attn_fwd_gqa(q, k, v, r=r, want_m=False)
    if plain:
        o, m = sb.sb_attn_fwd_train(q, k, v)
        return (o, m) + sb.sb_attn_bwd(q, k, v, m, s["dout"])
    o, m = sb.sb_attn_fwd_gqa(q, k, v, r=r)
    return (o, m) + sb.sb_attn_bwd_gqa(q, k, v, m, s["dout"], r=r)


def work(case):
    """A contraction is 2d operations per visible (query, key) pair: two forward, five backward.  For halt
    these are the full sweep's; how much of it the data lets a pass leave out is not in the sizes."""
    kind, B, H, Hkv, T, d = (case[n] for n in ("kind", "B", "H", "Hkv", "T", "d"))
    rows_q, rows_kv = B * H * T * d, B * Hkv * T * d
    if kind == "decode":
        return {"bytes": 4 * rows_kv + 4 * B * H * d, "flops": 4.0 * B * H * T * d}
    pairs = sum(n * (n - 1) // 2 for n in (lengths(case) if kind == "packed" else [T])) * B * H
    if kind == "f32":
        return {"bytes": 16 * rows_q, "flops": 4.0 * d * pairs}
    if kind in ("prefill", "halt"):
        return {"bytes": 4 * rows_q + 4 * rows_kv, "flops": 4.0 * d * pairs}
    # forward: q, k, v in, o and m out; backward: q, k, v, dout and m in, fp32 dq, dk, dv out
    return {"bytes": 12 * rows_q + 16 * rows_kv + 8 * B * H * T, "flops": 14.0 * d * pairs}


def tolerance(case):
    # fp32: sums over up to 2048 keys whose weights' exponents are themselves such sums.  bf16: weights and
    # dZ are rounded to bf16 before the second products, o is stored in bf16.
    return {"rel": 2e-5} if case["kind"] == "f32" else {"rel": 1e-2}
