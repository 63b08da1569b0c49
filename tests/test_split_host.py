"""The cut of the backward's key pass into row chunks and query-head parts: a
host build of the library's own rule (bwd_chunks), checked over 31 sequence
lengths x 4 batch sizes x 28 head layouts x 3 head dims, plain and under
AddressSanitizer and UndefinedBehaviorSanitizer (host code only); the
argument checks of basp_unpack_pack and its binding; and the order of a share's step."""
import ctypes
import os

import pytest
import torch

import paper_2609_03151_amd as basp
from paper_2609_03151_amd import share
from test_host_logic import HIPCC, SAN_ENV, SAN_HIPCC, _build_run


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
@pytest.mark.parametrize("sanitize", [False, True])
def test_bwd_plan(tmp_path, sanitize):
    out = _build_run(tmp_path, "bwd_plan_check.cpp", "bwd_plan_check",
                     SAN_HIPCC if sanitize else ["-O2"], env=SAN_ENV if sanitize else None)
    assert out.startswith("bwd plan ok")
    assert int(out.split()[-1]) == 31 * 4 * 28 * 3


def test_unpack_pack_checks_both_calls():
    """basp_unpack_pack reports what either of its two permutations would, before any launch."""
    L = basp.lib()
    tab = lambda base, n=2: (ctypes.c_void_p * n)(*[base + 0x1000 * j for j in range(n)])
    ok, none, f32, bf16 = 0, None, 1, 0
    call = lambda src, dst_t, src_t, dst, b=1, S=64, n=4, d=64, G=2, rank=0, dt=bf16: \
        L.basp_unpack_pack(src, dst_t, src_t, dst, b, S, n, d, G, rank, dt, none)
    a, t, u, c = 0x100000, tab(0x200000), tab(0x300000), 0x400000
    assert call(a, t, u, c, b=0) == ok                    # empty: no pointer is inspected
    assert call(none, none, none, none, S=0) == ok
    assert call(a, t, none, c) == 1 and call(a, none, u, c) == 1    # NULL
    assert call(none, t, u, c) == 1 and call(a, t, u, none) == 1
    assert call(a, t, (ctypes.c_void_p * 2)(0x1000, None), c) == 1
    assert call(a, t, u, c, S=63) == 2 and call(a, t, u, c, n=3) == 2   # SHAPE
    assert call(a, t, u, c, n=1) == 2                     # a shared head is not unpacked
    assert call(a, t, u, c, rank=2) == 3                  # RANK
    assert call(a, t, u, c, dt=7) == 4                    # UNSUPPORTED
    assert call(a, t, u, c + 1) == 5 and call(a + 2, t, u, c, dt=f32) == 5   # ALIGN


def test_unpack_pack_wants_as_many_sources_as_shards():
    mk = lambda n: [torch.zeros(1, 32, 4, 64) for _ in range(n)]
    local = torch.zeros(1, 64, 2, 64)
    for n in (1, 3):
        with pytest.raises(ValueError, match="number"):
            basp.unpack_pack(local, mk(2), mk(n), 0, out=torch.zeros_like(local))


def test_step_is_forward_then_backward(monkeypatch):
    """A step sends O before it takes dO, so that a dO that lives in O's send buffers (the loss
    half the sum of O squared) is the O of this step; and it goes through forward() and
    backward(), which a subclass may extend."""
    G, b, S, H, d = 2, 1, 8, 2, 64
    mk = lambda: [torch.zeros(b, S // G, H, d, dtype=torch.bfloat16) for _ in range(G)]

    def unpack(local, shards, rank):
        for j, t in enumerate(shards):
            t[:, :, rank] = local[:, j * S // G:(j + 1) * S // G, 0]

    def pack(shards, rank, out):
        out[:, :, 0] = torch.cat([t[:, :, rank] for t in shards], dim=1)

    both = lambda local, shards, src, rank, out: (pack(src, rank, out), unpack(local, shards, rank))
    for name, f in (("unpack", unpack), ("pack", pack), ("unpack_pack", both),
                    ("pack_qkv", lambda *a, **k: None), ("unpack_grads", lambda *a: None),
                    ("attn_fwd", lambda *a, out, **k: out.fill_(3.0)),
                    ("attn_bwd", lambda *a, **k: None)):
        monkeypatch.setattr(share, name, f, raising=False)
    sh = share.RankShare(mk(), mk(), mk(), None, G=G, rank=1)
    sh.do_shards = sh.o_shards
    sh.step()
    assert bool((sh.do == 3.0).all())

    seen = []

    class Traced(share.RankShare):
        def forward(self):
            seen.append("forward")
            super().forward()

        def pack_do(self):
            seen.append("pack_do")
            super().pack_do()

    Traced(mk(), mk(), mk(), mk(), G=G, rank=0).step()
    assert seen == ["forward", "pack_do"]
