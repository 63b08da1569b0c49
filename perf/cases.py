"""Timed cases: the calls a rank of a sequence-parallel group makes, over the range it makes them.

A case is one rank's share of the attention layer (b sequences of S tokens, H query and H_kv
key/value heads of dimension d, a group of G members, this rank's index), run in one of five ways:

  step      the composed share: pack Q, K, V -> attention -> unpack O, then pack dO -> backward ->
            unpack dQ, dK, dV (``RankShare.step``)
  in_place  the same step with attention on the exchange's shard buffers (``attn_fwd_sharded``,
            ``attn_bwd_sharded``; each tensor's G shards are one receive or send buffer)
  layer     attention forward and backward on head-sharded tensors (``attn_fwd``, ``attn_bwd``, or
            ``attn_bwd_noalloc`` when the case says so), as a program with its own exchange calls them
  receive   the rank's side of the exchanges alone: ``pack_qkv``, ``unpack`` of O, ``pack`` of dO,
            ``unpack_grads``
  owner     the sequence owner's side: ``a2a_pack`` of Q, K, V, ``a2a_unpack`` of O,
            ``a2a_pack_bf16`` of an fp32 dO, ``a2a_unpack`` of the fp32 gradients

Inputs are N(0, 1) activations in bf16 drawn on the GPU from the seed (fp32 for gradients).
``exact`` recomputes every output in plain fp64 torch.
"""
from __future__ import annotations

import math

import torch

import paper_2609_03151_amd as basp
from paper_2609_03151_amd.share import RankShare

BF16, F32, F64 = torch.bfloat16, torch.float32, torch.float64


def _case(name, kind, b, S, H, H_kv, d, G, rank, **more):
    c = {"kind": kind, "b": b, "S": S, "H": H, "H_kv": H_kv, "d": d, "G": G, "rank": rank, **more}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the smallest share: short sequences, small heads; launches and latency
        _case("tiny_step", "step", 2, 512, 8, 8, 64, 2, 0),
        # short training sequences, two per group, a group of 8: one kv head per rank
        _case("short_step_s2k", "step", 2, 2048, 32, 8, 128, 8, 3),
        # a ragged sequence, 7 query heads on one kv head, backward without a workspace argument
        _case("ragged_layer_s3k", "layer", 1, 3000, 28, 4, 128, 4, 2, noalloc=True),
        # an ordinary 8K context at Llama-3-8B shapes
        _case("llama3_8b_step_s8k", "step", 1, 8192, 32, 8, 128, 4, 1),
        # the 16K training setup at head dims 64, 96 and 80
        _case("llama32_1b_step_s16k", "step", 1, 16384, 32, 8, 64, 4, 3),
        _case("llama32_3b_in_place_s16k", "in_place", 1, 16384, 32, 8, 96, 4, 1),
        _case("qwen25_3b_layer_s16k", "layer", 1, 16384, 32, 8, 80, 4, 2, noalloc=False),
        # long contexts: the Llama-3-8B share at 32K, a kv head shared by two members at 64K
        _case("llama3_8b_step_s32k", "step", 1, 32768, 32, 8, 128, 4, 1),
        _case("llama3_8b_g16_in_place_s64k", "in_place", 1, 65536, 32, 8, 128, 16, 5),
        # the largest share one GPU takes: Llama-3-70B at 128K
        _case("llama3_70b_step_s128k", "step", 1, 131072, 64, 8, 128, 8, 5),
        # the exchange's permutations alone: the rank's side, and the owner's side with ragged
        # token counts and a head dim that is no power of two
        _case("receive_llama3_8b_s32k", "receive", 1, 32768, 32, 8, 128, 4, 1),
        _case("owner_d80_s12k", "owner", 2, 12012, 28, 4, 80, 4, 0),
    ]


# The most work a drawn case takes: below the largest listed one.
_MOST_FLOPS = 4e13
_MOST_ELEMS = 2 ** 28


def draw(rng):
    """One more share of the listed ranges: 256 to 64K tokens, 1 to 8 local query heads."""
    while True:
        kind = rng.choice(("step", "step", "in_place", "layer", "layer", "receive", "owner"))
        d = rng.choice((64, 80, 96, 128, 128))
        G = rng.choice((2, 4, 8))
        b = rng.choice((1, 1, 1, 2, 3))
        n_rep = rng.choice((1, 2, 4, 7, 8))
        Hkl = rng.choice((1, 1, 2, 4))
        H_kv = Hkl * G
        H = H_kv * n_rep
        if kind == "in_place" and Hkl == 1 and n_rep > 1 and rng.random() < 0.4:
            H_kv = G // 2  # a kv head shared by two members
        S = int(round(2.0 ** rng.uniform(8.0, 16.0)))
        unit = 256 * G if kind == "in_place" else G
        S = max(unit, S // unit * unit)
        if kind != "in_place" and rng.random() < 0.4:
            S += G * rng.randrange(1, 64)  # ragged: no multiple of any tile
        c = _case(None, kind, b, S, H, H_kv, d, G, rng.randrange(G))
        if kind == "layer":
            c["noalloc"] = b * Hkl * S <= 16384 and rng.random() < 0.5
        if Hkl * n_rep > 8 or work(c)["flops"] > _MOST_FLOPS or b * S * H * d > _MOST_ELEMS:
            continue
        return c


# ------------------------------------------------------------------ sizes
def _local_heads(c):
    return c["H"] // c["G"], max(1, c["H_kv"] // c["G"])


def work(c):
    b, S, d, G = c["b"], c["S"], c["d"], c["G"]
    Hl, Hkl = _local_heads(c)
    q, kv = b * S * Hl * d, b * S * Hkl * d  # elements of one local Q, of one local K
    if c["kind"] == "receive":  # bf16 Q, K, V, O, dO and fp32 dQ, dK, dV, each read and written
        return {"bytes": 2 * (2 * (3 * q + 2 * kv) + 4 * (q + 2 * kv)), "flops": 0}
    if c["kind"] == "owner":  # bf16 Q, K, V, O; fp32 dO to bf16; fp32 dQ, dK, dV
        oq, okv = b * (S // G) * c["H"] * d, b * (S // G) * c["H_kv"] * d
        return {"bytes": 2 * 2 * (2 * oq + 2 * okv) + 6 * oq + 2 * 4 * (oq + 2 * okv), "flops": 0}
    # bf16 Q, K, V, dO in; bf16 O, fp32 LSE, dQ, dK, dV out; causal half of seven S x S x d products
    return {"bytes": 2 * (3 * q + 2 * kv) + 4 * b * Hl * S + 4 * (q + 2 * kv),
            "flops": 3.5 * 2.0 * b * Hl * d * float(S) ** 2}


def tolerance(c):
    if c["kind"] in ("receive", "owner"):
        return "exact"
    # bf16 P and dS: 2.2e-3 relative and 0.26 of the rms at the worst element from fp64 at these
    # shapes, about four times of each
    return {"rel": 1e-2, "max": 0.9}


# ------------------------------------------------------------------ inputs
def _randn(gen, shape, dtype=BF16):
    return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)


def _inputs(c, seed):
    """The tensors a case starts from, drawn in a fixed order."""
    gen = torch.Generator("cuda").manual_seed(seed)
    b, S, H, H_kv, d, G = (c[k] for k in ("b", "S", "H", "H_kv", "d", "G"))
    Hl, Hkl = _local_heads(c)
    Sg = S // G
    if c["kind"] in ("step", "in_place"):  # G received shards of each
        shards = lambda n: [_randn(gen, (b, Sg, n, d)) for _ in range(G)]
        return {"q": shards(H), "k": shards(H_kv), "v": shards(H_kv), "do": shards(H)}
    if c["kind"] == "layer":
        return {"q": _randn(gen, (b, S, Hl, d)), "k": _randn(gen, (b, S, Hkl, d)),
                "v": _randn(gen, (b, S, Hkl, d)), "do": _randn(gen, (b, S, Hl, d))}
    if c["kind"] == "receive":
        shards = lambda n: [_randn(gen, (b, Sg, n, d)) for _ in range(G)]
        x = {"q": shards(H), "k": shards(H_kv), "v": shards(H_kv), "do": shards(H)}
        x["o"] = _randn(gen, (b, S, Hl, d))
        x["dq"], x["dk"], x["dv"] = (_randn(gen, (b, S, n, d), F32) for n in (Hl, Hkl, Hkl))
        return x
    x = {"q": _randn(gen, (b, Sg, H, d)), "k": _randn(gen, (b, Sg, H_kv, d)),
         "v": _randn(gen, (b, Sg, H_kv, d)), "do": _randn(gen, (b, Sg, H, d), F32)}
    x["o"] = _randn(gen, (G, b, Sg, Hl, d))
    x["dq"], x["dk"], x["dv"] = (_randn(gen, (G, b, Sg, n, d), F32) for n in (Hl, Hkl, Hkl))
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    b, S, H, H_kv, d, G, rank = (case[k] for k in ("b", "S", "H", "H_kv", "d", "G", "rank"))
    st = {"case": case, "x": x}
    if case["kind"] == "step":
        st["share"] = RankShare(x["q"], x["k"], x["v"], x["do"], G=G, rank=rank)
    elif case["kind"] == "in_place":
        buf = lambda n, t: torch.zeros((G, b, S // G, n, d), dtype=t, device="cuda")
        n_kv = H_kv if H_kv >= G else 1  # a shared kv head's gradients: one send block per member
        st["lse"] = torch.empty((b, H // G, S), dtype=F32, device="cuda")
        st["o"], st["dq"] = buf(H, BF16), buf(H, F32)
        st["dk"], st["dv"] = buf(n_kv, F32), buf(n_kv, F32)
        st["workspace"] = torch.empty(
            max(16, basp.attn_bwd_sharded_workspace_bytes(b, S, H, H_kv, d, G)),
            dtype=torch.uint8, device="cuda")
        st["shards"] = {n: list(st[n]) for n in ("o", "dq", "dk", "dv")}
    elif case["kind"] == "layer":
        if case["noalloc"]:
            st["grads"] = [torch.empty(x[n].shape, dtype=F32, device="cuda") for n in "qkv"]
        else:
            st["workspace"] = torch.empty(
                max(16, basp.attn_bwd_workspace_bytes(b, S, H, H_kv, d, G)), dtype=torch.uint8,
                device="cuda")
    elif case["kind"] == "receive":
        Hl, Hkl = _local_heads(case)
        local = lambda n: torch.empty((b, S, n, d), dtype=BF16, device="cuda")
        send = lambda n, t: [torch.zeros((b, S // G, n, d), dtype=t, device="cuda")
                             for _ in range(G)]
        st["q"], st["k"], st["v"], st["do"] = local(Hl), local(Hkl), local(Hkl), local(Hl)
        st["o_out"] = send(H, BF16)
        st["dq_out"], st["dk_out"], st["dv_out"] = send(H, F32), send(H_kv, F32), send(H_kv, F32)
    return st


# ------------------------------------------------------------------ one pass
def run(st):
    c, x = st["case"], st["x"]
    G, rank, H_kv = c["G"], c["rank"], c["H_kv"]
    if c["kind"] == "step":
        sh = st["share"]
        sh.step()
        return {"o": sh.o_shards, "lse": sh.lse, "dq": sh.dq_shards, "dk": sh.dk_shards,
                "dv": sh.dv_shards}
    if c["kind"] == "in_place":
        s = st["shards"]
        basp.attn_fwd_sharded(x["q"], x["k"], x["v"], s["o"], rank, lse=st["lse"])
        basp.attn_bwd_sharded(x["q"], x["k"], x["v"], s["o"], st["lse"], x["do"], s["dq"], s["dk"],
                              s["dv"], rank, workspace=st["workspace"])
        return {n: st[n] for n in ("o", "lse", "dq", "dk", "dv")}
    if c["kind"] == "layer":
        o, lse = basp.attn_fwd(x["q"], x["k"], x["v"], G=G, H_kv=H_kv)
        if c["noalloc"]:
            dq, dk, dv = basp.attn_bwd_noalloc(x["q"], x["k"], x["v"], o, lse, x["do"],
                                               *st["grads"], G=G, H_kv=H_kv)
        else:
            dq, dk, dv = basp.attn_bwd(x["q"], x["k"], x["v"], o, lse, x["do"], G=G, H_kv=H_kv,
                                       workspace=st["workspace"])
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    if c["kind"] == "receive":
        basp.pack_qkv(x["q"], x["k"], x["v"], rank, q=st["q"], k=st["k"], v=st["v"])
        basp.unpack(x["o"], st["o_out"], rank)
        basp.pack(x["do"], rank, out=st["do"])
        basp.unpack_grads(x["dq"], x["dk"], x["dv"], st["dq_out"], st["dk_out"], st["dv_out"],
                          rank)
        return {n: st[n] for n in ("q", "k", "v", "do", "o_out", "dq_out", "dk_out", "dv_out")}
    out = {n: basp.a2a_pack(x[n], G) for n in ("q", "k", "v")}
    out["o"] = basp.a2a_unpack(x["o"])
    out["do"] = basp.a2a_pack_bf16(x["do"], G)
    out["dq"] = basp.a2a_unpack(x["dq"])
    out["dk"] = basp.a2a_unpack(x["dk"], n_heads=H_kv)
    out["dv"] = basp.a2a_unpack(x["dv"], n_heads=H_kv)
    return out


# ------------------------------------------------------------------ fp64 reference
def _attention64(q, k, v, do, scale):
    """O, LSE, dQ, dK, dV of causal GQA attention in fp64, blockwise over query rows."""
    b, S, Hl, d = q.shape
    Hkl = k.shape[2]
    n_rep = Hl // Hkl
    new = lambda n: torch.zeros((b, S, n, d), dtype=F64, device=q.device)
    o, dq, dk, dv = new(Hl), new(Hl), new(Hkl), new(Hkl)
    lse = torch.empty((b, Hl, S), dtype=F64, device=q.device)
    for beta in range(b):
        for h in range(Hl):
            Q, dO = (t[beta, :, h].to(F64).contiguous() for t in (q, do))
            K, V = (t[beta, :, h // n_rep].to(F64).contiguous() for t in (k, v))
            block = max(256, min(4096, 2 ** 28 // S))
            for r0 in range(0, S, block):
                r1 = min(S, r0 + block)
                s = (Q[r0:r1] @ K[:r1].T) * scale
                s[:, r0:].masked_fill_(torch.ones(r1 - r0, r1 - r0, dtype=torch.bool,
                                                  device=q.device).triu_(1), -math.inf)
                l = torch.logsumexp(s, dim=1, keepdim=True)
                p = s.sub_(l).exp_()
                ob = p @ V[:r1]
                ds = (dO[r0:r1] @ V[:r1].T).sub_((dO[r0:r1] * ob).sum(1, keepdim=True)).mul_(p)
                dv[beta, :r1, h // n_rep] += p.T @ dO[r0:r1]
                dk[beta, :r1, h // n_rep] += scale * (ds.T @ Q[r0:r1])
                dq[beta, r0:r1, h] = scale * (ds @ K[:r1])
                o[beta, r0:r1, h], lse[beta, h, r0:r1] = ob, l[:, 0]
                del s, p, ds
    return o, lse, dq, dk, dv


def exact(case, seed):
    c = case
    b, S, H, H_kv, d, G, rank = (c[k] for k in ("b", "S", "H", "H_kv", "d", "G", "rank"))
    if work(c)["flops"] > 5e13:
        return None
    x = _inputs(c, seed)
    Hl, Hkl = _local_heads(c)
    Sg = S // G
    first = lambda n: rank * n // G
    if c["kind"] == "owner":
        split = lambda t, nl, n: torch.stack(
            [t[:, :, j * n // G:j * n // G + nl] for j in range(G)]).to(F64)
        join = lambda t: torch.cat(list(t.to(F64)), dim=2)
        return {"q": split(x["q"], Hl, H), "k": split(x["k"], Hkl, H_kv),
                "v": split(x["v"], Hkl, H_kv), "o": join(x["o"]), "do": split(x["do"], Hl, H),
                "dq": join(x["dq"]), "dk": join(x["dk"]), "dv": join(x["dv"])}
    cut = lambda ts, n, nl: torch.cat([t[:, :, first(n):first(n) + nl] for t in ts], dim=1)

    def spread(t, n):  # a local tensor in the rank's head slice of G shards, zeros elsewhere
        nl = t.shape[2]
        outs = [torch.zeros((b, Sg, n, d), dtype=F64, device=t.device) for _ in range(G)]
        for j, out in enumerate(outs):
            out[:, :, first(n):first(n) + nl] = t[:, j * Sg:(j + 1) * Sg].to(F64)
        return outs

    if c["kind"] == "receive":
        return {"q": cut(x["q"], H, Hl).to(F64), "k": cut(x["k"], H_kv, Hkl).to(F64),
                "v": cut(x["v"], H_kv, Hkl).to(F64), "do": cut(x["do"], H, Hl).to(F64),
                "o_out": spread(x["o"], H), "dq_out": spread(x["dq"], H),
                "dk_out": spread(x["dk"], H_kv), "dv_out": spread(x["dv"], H_kv)}
    scale = d ** -0.5
    if c["kind"] == "layer":
        o, lse, dq, dk, dv = _attention64(x["q"], x["k"], x["v"], x["do"], scale)
        return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
    q, k, v, do = cut(x["q"], H, Hl), cut(x["k"], H_kv, Hkl), cut(x["v"], H_kv, Hkl), cut(x["do"], H, Hl)
    o, lse, dq, dk, dv = _attention64(q, k, v, do, scale)
    if c["kind"] == "step":
        return {"o": spread(o, H), "lse": lse, "dq": spread(dq, H), "dk": spread(dk, H_kv),
                "dv": spread(dv, H_kv)}
    one = lambda t: torch.stack([t[:, j * Sg:(j + 1) * Sg] for j in range(G)])
    kv = one if H_kv < G else lambda t: torch.stack(spread(t, H_kv))
    return {"o": torch.stack(spread(o, H)), "lse": lse, "dq": torch.stack(spread(dq, H)),
            "dk": kv(dk), "dv": kv(dv)}
