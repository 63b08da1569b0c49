"""Parity of the attention when a row's maximum logit keeps growing.

The forward keeps, per query row, an exponent reference that starts at the
largest logit of the first keys and moves only when it has been outgrown;
moving it rescales the running sum, the output accumulator and, through them,
the LSE the backward uses.  It does so in two ways:

* where the maxima are formed (the kernel of small shares, whose waves each take
  32 keys of a tile with a reference of their own; diagonal tiles; the pipelined
  loop of short sequences), when a tile's maximum is more than 8 above it (in
  log2 units);
* in the pipelined loop of long sequences, when half a row's sum of a tile of 64
  keys has passed 2^16, for every row of the wave's 32.

With N(0,1) inputs at scale 1/sqrt(d) a row's maximum hardly grows after the
first tile, so these tests use ``ramped_local`` inputs, whose logits rise along
the sequence (Sec. II-A's softmax over long rows with a recency bias; the
incoming gradient dO at a quarter of unit scale keeps dK and dV, which such
concentrated attention enlarges, in the range of the other tests), and check,
from the inputs alone, that a stated share of (row, later tile) pairs, or of
moves per row, moves it by the rule of the kernel that runs.  O, LSE, dQ, dK and dV are then compared
element by element at the usual bar: small shapes, one of them with a key pass
of many row chunks, with the fp64 oracle, shapes past the small-share lines with
plain fp64 torch.
"""
import math

import pytest
import torch

import oracle
import paper_2609_03151_amd as basp
from parity import LSE_MAX_ABS, check_close, fp64_kv_head, log
from synth_inputs import ramped_local

pytestmark = pytest.mark.gpu

SLACK_LOG2 = 8.0    # a tile's maximum this far above the reference moves it
SUM_LOG2 = 16.0     # so does, in the pipelined loop, half a row's sum past 2 to this
WAVE_ROWS = 32      # rows of a wave, which move together there
RAMP = 24.0         # twice the rise of the other cases' logits: two moves in a long row


def _logits(q, k, scale, beta, h, n_rep, keys):
    """Causal logits of one head in log2 units, fp64, padded with -inf to ``keys`` columns."""
    S = q.shape[1]
    s = torch.full((S, keys), float("-inf"), dtype=torch.float64, device=q.device)
    s[:, :S] = (q[beta, :, h].double() @ k[beta, :, h // n_rep].double().T) * (scale / math.log(2.0))
    rows = torch.arange(S, device=q.device)
    return s.masked_fill_(torch.arange(keys, device=q.device)[None, :] > rows[:, None],
                          float("-inf"))


def _by_maxima(s, parts):
    """(moves, pairs, moves of each row): key parts of 32 keys, each with its reference."""
    S = s.shape[0]
    tmax = s.reshape(S, -1, parts, 32).max(dim=3).values  # [row, tile, part]
    ref = tmax[:, 0].clone()
    count = torch.zeros(S, dtype=torch.int64, device=s.device)
    pairs = 0
    for t in range(1, tmax.shape[1]):
        m = tmax[:, t]
        later = torch.isfinite(m) & torch.isfinite(ref)
        grow = later & (m > ref + SLACK_LOG2)
        count += grow.sum(1)
        pairs += int(later.sum())
        ref = torch.where(grow | ~torch.isfinite(ref), m, ref)
    return int(count.sum()), pairs, count


def _by_sums(s, parts):
    """The same in the pipelined loop: workgroups of 256 / parts rows, parts of 64 keys, the
    tiles left of a workgroup's diagonal band."""
    S, tile = s.shape[0], 64 * parts
    rows = 256 // parts
    # Lane l and l + 32 of a row hold keys 0-3 and 4-7 of every 8.
    x = s.reshape(S, -1, parts, 8, 2, 4)
    ref = x[:, 0].amax(dim=(2, 3, 4))  # [row, part]
    q0 = torch.arange(S, device=s.device) // rows * rows
    wave = torch.arange(S, device=s.device) // WAVE_ROWS
    count = torch.zeros(S, dtype=torch.int64, device=s.device)
    pairs = 0
    for t in range(1, S // tile):
        live = (t * tile < q0)[:, None]
        up = torch.log2(torch.exp2(x[:, t] - ref[:, :, None, None, None]).sum(dim=(2, 4)).amax(2))
        own = live & (up > SUM_LOG2)
        together = torch.zeros((int(wave[-1]) + 1, parts), dtype=torch.int32, device=s.device)
        together = together.index_add_(0, wave, own.int()) > 0
        moved = live & together[wave] & (up > 0.0)
        ref = torch.where(moved, ref + up, ref)
        count += moved.sum(1)
        pairs += int(live.sum()) * parts
    return int(count.sum()), pairs, count


def reference_moves(q, k, scale, rule, parts):
    """(moves, pairs, rows moved twice or more) over every (sequence, head, row)."""
    b, S, Hl, _ = q.shape
    keys = (S + 127) // 128 * 128
    total = [0, 0, 0]
    for beta in range(b):
        for h in range(Hl):
            moves, pairs, count = rule(_logits(q, k, scale, beta, h, Hl // k.shape[2], keys), parts)
            total = [total[0] + moves, total[1] + pairs, total[2] + int((count >= 2).sum())]
    return total


CASES = [  # b, S, Hl, Hkl, d, least fraction of (row, later tile) pairs that move
    (1, 1000, 4, 2, 128, 0.05),   # ragged tail, GQA 2 (15% move)
    (2, 777, 2, 1, 64, 0.10),     # d = 64, b = 2, ragged (31%)
    (1, 1200, 3, 1, 96, 0.05),    # d = 96, GQA 3 (17%)
    (1, 4096, 4, 1, 128, 0.015),  # key pass in eight row chunks, GQA 4 (4.4%)
]


@pytest.mark.parametrize("b,S,Hl,Hkl,d,frac", CASES)
def test_moving_reference_matches_oracle(b, S, Hl, Hkl, d, frac):
    log(f"[rescale] b={b} S={S} Hl={Hl} Hkl={Hkl} d={d}")
    q, k, v, do = ramped_local(b, S, Hl, Hkl, d, seed=S + d)
    scale = 1.0 / math.sqrt(d)
    qd, kd, vd, dod = (x.cuda() for x in (q, k, v, do))
    moves, pairs, multi = reference_moves(qd, kd, scale, _by_maxima, 4)
    log(f"  reference moves: {moves} of {pairs} (row, later tile) pairs "
        f"({moves / pairs:.3%}); rows moved at least twice: {multi}")
    assert moves >= frac * pairs, "inputs do not exercise the moving reference"
    assert multi > 0
    o, lse = basp.attn_fwd(qd, kd, vd, G=1, scale=scale)
    dq, dk, dv = basp.attn_bwd(qd, kd, vd, o, lse, dod, G=1, scale=scale)
    torch.cuda.synchronize()
    ro, rl = oracle.attn_fwd(q, k, v, scale)
    rdq, rdk, rdv = oracle.attn_bwd(q, k, v, do, ro, rl, scale)
    f64 = lambda t: t.double().cpu().numpy()
    check_close("O", f64(o), ro)
    check_close("LSE", f64(lse), rl, max_abs=LSE_MAX_ABS, mean_abs=LSE_MAX_ABS)
    check_close("dQ", f64(dq), rdq)
    check_close("dK", f64(dk), rdk)
    check_close("dV", f64(dv), rdv)


LONG = [  # b, S, Hl, Hkl, d, key parts of a workgroup
    (1, 5120, 8, 2, 128, 2), (2, 3600, 6, 2, 80, 2), (1, 8200, 6, 1, 96, 2),  # 128 rows
    (4, 3400, 8, 2, 64, 1), (4, 5000, 5, 1, 80, 1), (4, 5000, 5, 5, 96, 1),   # 256 rows
    (3, 7200, 4, 1, 128, 1),
]


@pytest.mark.parametrize("b,S,Hl,Hkl,d,parts", LONG)
def test_reference_that_follows_the_sums(b, S, Hl, Hkl, d, parts):
    log(f"[rescale sums] b={b} S={S} Hl={Hl} Hkl={Hkl} d={d}")
    q, k, v, do = (x.cuda() for x in ramped_local(b, S, Hl, Hkl, d, seed=S + d, ramp=RAMP,
                                                     do_std=0.125))
    scale = 1.0 / math.sqrt(d)
    moves, pairs, multi = reference_moves(q, k, scale, _by_sums, parts)
    rows = b * Hl * S
    log(f"  reference moves: {moves} of {pairs} (row, later tile) pairs, {moves / rows:.3f} a row; "
        f"rows moved at least twice: {multi / rows:.3f}")
    assert moves >= 0.5 * rows and multi >= 0.2 * rows, "the reference is not exercised"
    o, lse = basp.attn_fwd(q, k, v, scale=scale)
    dq, dk, dv = basp.attn_bwd(q, k, v, o, lse, do, scale=scale)
    torch.cuda.synchronize()
    n = Hl // Hkl
    f64 = lambda t: t.double().cpu().numpy()
    for beta in range(b):
        at = slice(beta, beta + 1)
        for h in range(Hkl):
            hq, hk = slice(h * n, (h + 1) * n), slice(h, h + 1)
            ref = fp64_kv_head(q[at, :, hq], k[at, :, hk], v[at, :, hk], do[at, :, hq], n, scale)
            got = o[beta, :, hq], dq[beta, :, hq], dk[beta, :, h], dv[beta, :, h]
            for name, x, want in zip(("O", "dQ", "dK", "dV"), got, ref):
                check_close(name, f64(x), f64(want))
            for g in range(h * n, (h + 1) * n):
                s = _logits(q, k, scale, beta, g, n, S) * math.log(2.0)
                check_close("LSE", f64(lse[beta, g]), f64(torch.logsumexp(s, dim=1)),
                            max_abs=LSE_MAX_ABS, mean_abs=LSE_MAX_ABS)


def test_moving_reference_in_place_path_is_bitwise_the_same():
    """The in-place forward (shard buffers, G = 4) on ramped inputs gives the
    composed path's O and LSE bit for bit."""
    b, S, Hl, Hkl, d, G, rank = 1, 2048, 2, 1, 128, 4, 1
    q, k, v, do = ramped_local(b, S, Hl * G, Hkl * G, d, seed=99)
    scale = 1.0 / math.sqrt(d)
    chunks = lambda x: [c.contiguous().cuda() for c in torch.chunk(x, G, dim=1)]
    qs, ks, vs = chunks(q), chunks(k), chunks(v)
    o_sh = [torch.zeros_like(s) for s in qs]
    lse_a = basp.attn_fwd_sharded(qs, ks, vs, o_sh, rank, scale=scale)
    ql = basp.pack(qs, rank)
    kl, vl = basp.pack(ks, rank), basp.pack(vs, rank)
    o, lse_b = basp.attn_fwd(ql, kl, vl, G=G, scale=scale, H_kv=Hkl * G)
    torch.cuda.synchronize()
    o_cat = torch.cat([s[:, :, rank * Hl:(rank + 1) * Hl] for s in o_sh], dim=1)
    assert torch.equal(o_cat.view(torch.int16), o.view(torch.int16))
    assert torch.equal(lse_a, lse_b)
