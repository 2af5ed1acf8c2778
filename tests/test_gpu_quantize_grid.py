"""The quantizer's grid: capacities far beyond use, and 16-bit rows in groups (needs an MI355X)."""
import numpy as np
import pytest

from paper_2605_02262_amd import synth
from tests.test_gpu_parity import _check, _custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("room", [0, 64])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16, synth.F32])
@pytest.mark.parametrize("Hkv", [1, 3])
def test_capacities_and_groups_of_rows(Hkv, dtype, room):
    """Capacities that just fit (blocks numbered by capacity) and that hold more than all rows fill (numbered by use), with every
    class empty in some sequence; 1, 7, 8 and 9 rows of 16 bits at the end of a sequence, windows among them (top tier of 16 bits)."""
    from tests import wq_harness as H
    for top_bits in (8, 16):
        specs = [synth.SeqSpec(9, 21, 21, 8, (2, 3, 4)), synth.SeqSpec(3, 16, 16, 1, (0, 1, 2)), synth.SeqSpec(0, 10, 4, 7, (0, 0, 0)),
                 synth.SeqSpec(4, 33, 33, 9, (4, 0, 0), tail=2), synth.SeqSpec(2, 32, 32, 0, (0, 0, 2))]
        bt = _custom(40 + Hkv + dtype + top_bits, 64, 32, Hkv, 2, dtype, specs, top_bits=top_bits, pin=0)
        cap, off16 = H.capacities(bt.w, slack=2)
        g, _, _ = _check(bt, H, cap=[c + 32 * room * (k + 1) for k, c in enumerate(cap)], off16=off16, splits=2)
        assert g.ctx.device_status() == 0


def test_more_blocks_than_a_grid_dimension():
    """44 000 sequences of one 2-bit token and two 16-bit rows, 128 KV heads, room for three blocks of each: one workgroup per
    block and head is more than one dimension of a launch takes, and the 16-bit rows come last.  Same rows as without the room."""
    import torch
    from paper_2605_02262_amd import binding as W
    B, Hkv, hd = 44000, 128, 64
    i32 = lambda x: torch.as_tensor(np.asarray(x, np.int32)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(11)
    K, V = (torch.randn(3 * B, Hkv, hd, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    kv_off, win_off, win_size = i32(3 * np.arange(B + 1)), i32(np.arange(B + 1)), i32(np.ones(B))
    ctx = W.Context(W.workspace_bytes(B, Hkv, hd, 1))
    quota = i32(np.tile([0, 0, 1], (B, 1)))
    bits, perm, seg = W.wq_assign_bits(ctx, torch.zeros(B, device="cuda"), win_off, 1, W.MODE_QUOTA, quota, None, 8, 0)
    rows = K.view(B, 3, Hkv, hd)[:, 1:].reshape(-1, Hkv, hd), V.view(B, 3, Hkv, hd)[:, 1:].reshape(-1, Hkv, hd)
    seen = []
    for room in (1, 3):
        pk = W.PackedKV(B, Hkv, hd, 64, torch.bfloat16, [32 * B * room, 0, 0], 2 * np.arange(B + 1))
        W.wq_reorder_quantize(ctx, K, V, kv_off, win_size, win_off, perm, seg, 3 * B, pk)
        assert ctx.device_status() == 0
        assert bool((pk.len16 == 2).all()) and bool((pk.cls_len[0] == 1).all())
        assert torch.equal(pk.k16, rows[0]) and torch.equal(pk.v16, rows[1]), room
        # the one code of every row: first token of a K tile, in use whatever the room
        seen.append(pk.meta[0].view(2, Hkv, B * room, 32)[:, :, :B, 0].clone())
    assert torch.equal(seen[0], seen[1])
