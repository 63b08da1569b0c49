"""GPU parity at the sizes where the work of a small share is cut finer, every
output against a plain fp64 torch computation on the GPU.

The backward's key pass is cut into row chunks and query-head parts (several
partial sums of dK and dV per key): uneven parts, ragged lengths, parts with
one chunk, chunks with one part, b > 1, each head dim.  Its dQ pass gives a
workgroup 256, 128 or 64 query rows by the share's rows (b * Hl * S): each
width on both sides of its lines, ragged and shorter than one tile.  The
forward gives a workgroup 256, 128 or 64 query rows likewise; each width is also
run on scores that grow or jump along the sequence (running references that
move, key parts of very different weight, P past the range of fp32 until the
reference has followed), on rows most key parts never reach, and in place on
the shard buffers."""
import math

import pytest
import torch

import paper_2609_03151_amd as basp
from paper_2609_03151_amd.share import RankShare
from parity import LSE_MAX_ABS, MAX_ABS, check_close, fp64_kv_head, log

pytestmark = pytest.mark.gpu

CASES = [  # b, S, Hl, Hkl, d
    (1, 1024, 8, 1, 128),   # 4 chunks x 4 parts
    (1, 1100, 7, 1, 96),    # 5 chunks x 4 parts of 1 and 2 heads, ragged
    (2, 2048, 4, 1, 128),   # 8 chunks, b = 2
    (1, 3000, 7, 1, 128),   # 12 chunks, ragged
    (3, 769, 6, 2, 80),     # the last key tile one key long
    (1, 2113, 3, 3, 64),    # chunks only
    (1, 6000, 10, 2, 64),   # long ragged chunks
    (1, 8192, 8, 2, 64),    # key units before dQ tiles, 2 chunks
    (1, 8192, 8, 8, 64),    # one unit per key tile
    (2, 9000, 10, 2, 128),  # 2 chunks x 2 parts
    (1, 11008, 20, 1, 64),  # parts of unlike size (6 and 7 heads)
    # dQ rows per workgroup: 64, then 128, then 256
    (1, 1, 1, 1, 128), (1, 63, 2, 1, 64), (1, 65, 1, 1, 96), (2, 129, 3, 3, 128),
    (1, 4608, 4, 2, 64), (1, 9216, 2, 1, 128),
    (1, 4609, 4, 2, 128), (3, 1500, 6, 2, 96), (1, 4097, 8, 4, 80),
    (2, 2304, 8, 2, 128), (2, 2305, 8, 2, 128),
    # forward rows per workgroup: 64 | 128 and 128 | 256
    (1, 4800, 8, 2, 128), (1, 4801, 8, 2, 96), (1, 10240, 8, 2, 80), (1, 10241, 8, 2, 80),
    (2, 6656, 8, 4, 64), (2, 6657, 8, 4, 64), (160, 130, 4, 2, 128), (300, 128, 1, 1, 96),
    # many short sequences: 256, 128 and 64 rows by how often they fill the GPU
    (8, 512, 4, 2, 128), (33, 512, 1, 1, 128), (65, 512, 1, 1, 80), (35, 257, 4, 1, 96),
    (188, 129, 1, 1, 64), (189, 128, 1, 1, 64), (50, 200, 4, 4, 64), (22, 1024, 1, 1, 96),
]


def _reference(q, k, v, do, scale):
    """O, LSE, dQ, dK, dV in fp64, one kv head of one sequence at a time."""
    b, S, Hl, d = q.shape
    n = Hl // k.shape[2]
    out = [torch.empty(t.shape, dtype=torch.float64, device="cuda") for t in (q, q, k, k)]
    lse = torch.empty((b, Hl, S), dtype=torch.float64, device="cuda")
    for beta in range(b):
        for h in range(k.shape[2]):
            hq, hk = slice(h * n, (h + 1) * n), slice(h, h + 1)
            at = slice(beta, beta + 1)
            args = q[at, :, hq], k[at, :, hk], v[at, :, hk], do[at, :, hq]
            o, dq, dk, dv = fp64_kv_head(*args, n, scale)
            out[0][beta, :, hq], out[1][beta, :, hq] = o, dq
            out[2][beta, :, h], out[3][beta, :, h] = dk, dv
            K = k[beta, :, h].double()
            for g in range(h * n, (h + 1) * n):
                for r0 in range(0, S, 2048):
                    r1 = min(S, r0 + 2048)
                    s = (q[beta, r0:r1, g].double() @ K[:r1].T) * scale
                    s[:, r0:].masked_fill_(torch.ones(r1 - r0, r1 - r0, dtype=torch.bool,
                                                      device="cuda").triu_(1), -math.inf)
                    lse[beta, g, r0:r1] = torch.logsumexp(s, dim=1)
    return out[0], lse, out[1], out[2], out[3]


@pytest.mark.parametrize("b,S,Hl,Hkl,d", CASES)
def test_split_attention_matches_fp64(b, S, Hl, Hkl, d):
    log(f"[split] b={b} S={S} Hl={Hl} Hkl={Hkl} d={d}")
    g = torch.Generator("cuda").manual_seed(S + 31 * Hl + d)
    mk = lambda n: torch.randn((b, S, n, d), generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, do = mk(Hl), mk(Hkl), mk(Hkl), mk(Hl)
    scale = d ** -0.5
    o, lse = basp.attn_fwd(q, k, v, scale=scale)
    need = basp.attn_bwd_workspace_bytes(b, S, Hl, Hkl, d, 1)
    # NaN everywhere the backward writes: nothing may be left out, and nothing
    # of the workspace is read before it is written.
    ws = torch.full(((need + 3) // 4,), math.nan, dtype=torch.float32, device="cuda")
    grads = [torch.full(t.shape, math.nan, dtype=torch.float32, device="cuda") for t in (q, k, v)]
    dq, dk, dv = basp.attn_bwd(q, k, v, o, lse, do, scale=scale, dq=grads[0], dk=grads[1],
                               dv=grads[2], workspace=ws)
    torch.cuda.synchronize()
    ref = _reference(q, k, v, do, scale)
    f = lambda t: t.double().cpu().numpy()
    # The bar on a key's dK and dV holds for up to 8 query heads on a kv head.
    # Each head adds its own rounding of bf16 P and dS, independent of the
    # others', so beyond 8 the sum's error grows with the root of their number.
    kv_bar = MAX_ABS * max(1.0, (Hl / Hkl / 8) ** 0.5)
    bars = {"LSE": dict(max_abs=LSE_MAX_ABS, mean_abs=LSE_MAX_ABS),
            "dK": dict(max_abs=kv_bar), "dV": dict(max_abs=kv_bar)}
    for name, got, want in zip(("O", "LSE", "dQ", "dK", "dV"), (o, lse, dq, dk, dv), ref):
        bar = bars.get(name, {})
        check_close(name, f(got), f(want), **bar)


@pytest.mark.parametrize("b,S,Hl,Hkl,d", [
    (1, 1000, 4, 1, 128), (2, 700, 2, 2, 64),   # 64 rows per workgroup
    (1, 5000, 8, 1, 128), (1, 5000, 8, 1, 80),  # 128
    (8, 2000, 7, 1, 64), (8, 2000, 7, 1, 80), (8, 2000, 7, 1, 96), (8, 2000, 7, 1, 128),  # 256
    # sequences long enough for the loop without row maxima: 128 rows, then 256
    (1, 9000, 8, 1, 96), (4, 7000, 5, 1, 64), (4, 7000, 5, 1, 80), (4, 7000, 5, 1, 96),
    (4, 7000, 5, 1, 128),
])
@pytest.mark.parametrize("peak", ["late", "early", "jumps"])
def test_forward_references_that_move(b, S, Hl, Hkl, d, peak):
    """Scores that rise (or fall) along the keys by tens of units, or jump by
    hundreds at single keys (exp2 of the difference is past fp32's range): each
    running reference moves many times, and a row's key parts differ in weight
    by many orders of magnitude when they are merged."""
    log(f"[split ramp] b={b} S={S} Hl={Hl} Hkl={Hkl} d={d} {peak}")
    g = torch.Generator("cuda").manual_seed(S + d)
    mk = lambda n: torch.randn((b, S, n, d), generator=g, device="cuda")
    q, k, v, do = mk(Hl), mk(Hkl), mk(Hkl), mk(Hl)
    ramp = torch.linspace(0, 40, S, device="cuda")[None, :, None]
    if peak == "jumps":  # 0 but for a handful of keys, each 150 above the one before
        ramp = torch.zeros_like(ramp)
        for i, at in enumerate((70, S // 5, S // 2 + 1, 3 * S // 4, S - 100)):
            ramp[:, at] = 150.0 * (i + 1)
    q[..., 0], k[..., 0] = d ** 0.25, (-ramp if peak == "early" else ramp) * d ** 0.25
    q, k, v, do = (t.to(torch.bfloat16) for t in (q, k, v, do))
    o, lse = basp.attn_fwd(q, k, v)
    ref = _reference(q, k, v, do, d ** -0.5)
    f = lambda t: t.double().cpu().numpy()
    check_close("O", f(o), f(ref[0]))
    check_close("LSE", f(lse), f(ref[1]), max_abs=LSE_MAX_ABS, mean_abs=LSE_MAX_ABS)


@pytest.mark.parametrize("b,S,Hl,d", [
    *((8, 1024, 8, d) for d in (64, 128)), *((8, 2048, 7, d) for d in (64, 128)),  # row maxima
    *((8, 3584, 2, d) for d in (80, 96, 128)),      # row sums, 128 rows
    *((8, 6656, 3, d) for d in (64, 80, 96, 128)),  # row sums, 256 rows
])
def test_forward_jump_near_the_top_of_fp32(b, S, Hl, d):
    """One key 87 to 89 units (126 to 128 powers of two) above the row's reference: P is finite
    and so are its sums, but the factor that brings them to the new reference is below fp32's
    normal range.  Keys 0 .. 127 score 0 exactly, so every row of a sequence jumps by the same
    amount; a later key scores 1.4 below the jump.  The shards in place give the same bits."""
    log(f"[split jump] b={b} S={S} Hl={Hl} d={d}")
    G, rank = 2, 1
    g = torch.Generator("cuda").manual_seed(S + d)
    mk = lambda n: torch.randn((b, S, n, d), generator=g, device="cuda")
    q, k, v, do = mk(Hl), mk(1), 0.25 * mk(1), mk(Hl)
    k[:, :128] = 0.0
    scale = 0.125
    q[..., :2], k[..., :2] = 8.0, 0.0  # times the scale: a key's first two elements are its score
    for beta, jump in enumerate((87.0, 87.4, 87.6, 88.0, 88.4, 88.6, 88.7, 89.0)):
        for at, score in ((300, jump), (700, jump - 1.4)):
            k[beta, at] = 0.0
            k[beta, at, 0, 0] = score
            k[beta, at, 0, 1] = score - float(torch.tensor(score).bfloat16())
    q, k, v, do = (t.to(torch.bfloat16) for t in (q, k, v, do))
    o, lse = basp.attn_fwd(q, k, v, scale=scale)
    other = lambda t: torch.cat([torch.zeros_like(t), t], dim=2)  # rank 0's heads, rank 1's
    shards = lambda t: [x.contiguous() for x in torch.chunk(other(t), G, dim=1)]
    q_sh, k_sh, v_sh = shards(q), shards(k), shards(v)
    o_sh = [torch.zeros_like(t) for t in q_sh]
    lse_sh = basp.attn_fwd_sharded(q_sh, k_sh, v_sh, o_sh, rank, scale=scale)
    torch.cuda.synchronize()
    ref = _reference(q, k, v, do, scale)
    f = lambda t: t.double().cpu().numpy()
    check_close("O", f(o), f(ref[0]))
    check_close("LSE", f(lse), f(ref[1]), max_abs=LSE_MAX_ABS, mean_abs=LSE_MAX_ABS)
    got = torch.cat([t[:, :, Hl:] for t in o_sh], dim=1)
    assert torch.equal(got.view(torch.int16), o.view(torch.int16))
    assert torch.equal(lse_sh, lse)


@pytest.mark.parametrize("b,S,Hl,Hkl,d,share", [
    (1, 3000, 8, 2, 128, 0.55), (1, 3000, 8, 2, 128, 0.3), (1, 1024, 8, 1, 128, 0.6),
    (2, 2048, 4, 1, 128, 0.5), (1, 1500, 8, 2, 128, 0.0), (2, 4100, 4, 1, 96, 0.0),
])
def test_backward_in_a_small_workspace(b, S, Hl, Hkl, d, share):
    """A workspace below the size the query reports (the least, and between): the cut fits it,
    nothing past its end is written, and the gradients hold."""
    g = torch.Generator("cuda").manual_seed(S + d)
    mk = lambda n: torch.randn((b, S, n, d), generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, do = mk(Hl), mk(Hkl), mk(Hkl), mk(Hl)
    rows = max(2048, min(8192, S // 4 // 128 * 128))
    least = 8 * b * Hl * ((S + 63) // 64 * 64)  # the planes, then one sum per row chunk
    if S > rows:
        least = (least + 255) // 256 * 256 + 8 * b * S * Hkl * d * ((S + rows - 1) // rows)
    need = basp.attn_bwd_workspace_bytes(b, S, Hl, Hkl, d, 1)
    n = (least + int(share * (need - least))) // 16 * 16
    log(f"[split workspace] b={b} S={S} Hl={Hl} Hkl={Hkl} d={d}: {n} of {need} bytes")
    assert n < need
    o, lse = basp.attn_fwd(q, k, v)
    ws = torch.full((need // 4 + 64,), math.nan, dtype=torch.float32, device="cuda")
    ws[n // 4:] = 7.0
    grads = [torch.full(t.shape, math.nan, dtype=torch.float32, device="cuda") for t in (q, k, v)]
    basp.attn_bwd(q, k, v, o, lse, do, dq=grads[0], dk=grads[1], dv=grads[2],
                  workspace=ws[:n // 4])
    torch.cuda.synchronize()
    assert bool((ws[n // 4:] == 7.0).all())
    _, _, *ref = _reference(q, k, v, do, d ** -0.5)
    for name, got, want in zip(("dQ", "dK", "dV"), grads, ref):
        check_close(name, got.double().cpu().numpy(), want.cpu().numpy())


def test_backward_of_more_workgroups_than_one_launch_takes():
    """65535 sequences of one token, 65 heads: each pass fits a launch, both together do not.
    With one key P = 1, so O = V and dV = dO bit for bit, and dQ = dK = 0 up to rounding."""
    b, H, d = 65535, 65, 64
    log(f"[split launches] b={b} S=1 H={H} d={d}")
    g = torch.Generator("cuda").manual_seed(1)
    q, k, v, do = (torch.randn((b, 1, H, d), generator=g, device="cuda", dtype=torch.bfloat16)
                   for _ in range(4))
    o, lse = basp.attn_fwd(q, k, v)
    grads = [torch.full(t.shape, math.nan, dtype=torch.float32, device="cuda") for t in (q, k, v)]
    basp.attn_bwd(q, k, v, o, lse, do, dq=grads[0], dk=grads[1], dv=grads[2])
    torch.cuda.synchronize()
    assert torch.equal(o, v) and torch.equal(grads[2], do.float())
    assert max(float(t.abs().max()) for t in grads[:2]) <= MAX_ABS


@pytest.mark.parametrize("b,S,n,d,G,dtype", [
    (2, 512, 8, 64, 2, torch.bfloat16), (1, 96, 6, 3, 3, torch.bfloat16),  # 16- and 2-byte rows
    (1, 340, 17, 20, 17, torch.float32), (1, 8192, 32, 128, 8, torch.bfloat16),  # G > 16: two launches
])
def test_unpack_pack_is_both_calls(b, S, n, d, G, dtype):
    g = torch.Generator("cuda").manual_seed(S)
    mk = lambda: [torch.randn((b, S // G, n, d), generator=g, device="cuda").to(dtype)
                  for _ in range(G)]
    src, rank = mk(), G - 1
    local = torch.randn((b, S, n // G, d), generator=g, device="cuda").to(dtype)
    want = basp.unpack(local, [torch.zeros_like(t) for t in src], rank)
    got, out = [torch.zeros_like(t) for t in src], torch.empty_like(local)
    basp.unpack_pack(local, got, src, rank, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, basp.pack(src, rank))
    assert all(torch.equal(x, y) for x, y in zip(got, want))


def test_shards_from_an_iterator():
    """The tables of V and of dV may come from iterators, which are walked once."""
    G, rank = 2, 1
    g = torch.Generator("cuda").manual_seed(4)
    mk = lambda h, t: [torch.randn((1, 64, h, 64), generator=g, device="cuda").to(t) for _ in range(G)]
    q, k, v = mk(4, torch.bfloat16), mk(2, torch.bfloat16), mk(2, torch.bfloat16)
    assert all(torch.equal(a, c) for a, c in zip(basp.pack_qkv(q, k, iter(v), rank),
                                                 basp.pack_qkv(q, k, v, rank)))
    local = [torch.cat(t, dim=1)[:, :, :n].contiguous().float() for t, n in ((q, 2), (k, 1), (v, 1))]
    want, got = ([mk(h, torch.float32) for h in (4, 2, 2)] for _ in range(2))
    for w, x in zip(want, got):
        for a, c in zip(w, x):
            c.copy_(a)
    basp.unpack_grads(*local, *want, rank)
    basp.unpack_grads(*local, got[0], got[1], iter(got[2]), rank)
    torch.cuda.synchronize()
    assert all(torch.equal(a, c) for w, x in zip(want, got) for a, c in zip(w, x))


def test_step_with_d_o_in_the_send_buffers():
    """dO = O in place (the loss half the sum of O squared): a step is forward(), then backward()."""
    G, b, S, n, d, rank = 2, 1, 1024, 4, 64, 1
    g = torch.Generator("cuda").manual_seed(3)
    mk = lambda h: [torch.randn((b, S // G, h, d), generator=g, device="cuda").to(torch.bfloat16)
                    for _ in range(G)]
    q, k, v = mk(2 * n), mk(2), mk(2)
    want, got = (RankShare(q, k, v, None, G=G, rank=rank) for _ in range(2))
    for sh in (want, got):
        sh.do_shards = sh.o_shards
    want.forward()
    torch.cuda.synchronize()
    want.backward()
    got.step()
    torch.cuda.synchronize()
    assert torch.equal(got.do, got.o) and bool(got.o.any())
    for name in ("dq_shards", "dk_shards", "dv_shards"):
        assert all(torch.equal(a, c) for a, c in zip(getattr(got, name), getattr(want, name)))


@pytest.mark.parametrize("S", [1024, 5120, 16384])
@pytest.mark.parametrize("d", [64, 128])
def test_split_forward_in_place(S, d):
    """The three workgroup widths read the shards as they read local tensors."""
    G, b, n, rank = 2, 1, 8, 1
    g = torch.Generator("cuda").manual_seed(S + d)
    mk = lambda h: [torch.randn((b, S // G, h, d), generator=g, device="cuda").to(torch.bfloat16)
                    for _ in range(G)]
    q, k, v = mk(2 * n), mk(2), mk(2)
    o_sh = [torch.zeros_like(t) for t in q]
    lse_sh = basp.attn_fwd_sharded(q, k, v, o_sh, rank)
    local = basp.pack_qkv(q, k, v, rank)
    o, lse = basp.attn_fwd(*local, G=G)
    torch.cuda.synchronize()
    got = torch.cat([t[:, :, rank * n:(rank + 1) * n] for t in o_sh], dim=1)
    assert torch.equal(got.view(torch.int16), o.view(torch.int16))
    assert torch.equal(lse_sh, lse)
