"""Tensors that do not begin on a 16-byte boundary: cut out of larger ones (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth

pytestmark = pytest.mark.gpu


def _off_by_one(t):
    """The same values one element behind a 16-byte boundary."""
    room = torch.empty(t.numel() + 8, dtype=t.dtype, device=t.device)
    room[1:1 + t.numel()] = t.reshape(-1)
    got = room[1:1 + t.numel()].view(t.shape)
    assert got.data_ptr() % 16 == t.element_size()
    return got


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16, synth.F32])
@pytest.mark.parametrize("hd,g", [(128, 32), (128, 128), (64, 64)])
def test_one_and_four_groups_take_any_alignment(hd, g, dtype):
    """Query, appended rows and 16-bit segment one element off: what the vector kernel and the append kernel take.  The 16-bit
    rows are written off the boundary by the quantizer as well."""
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    from tests.test_gpu_decode_groups import TIGHT
    dt16 = synth.BF16 if dtype == synth.BF16 else synth.F16
    specs = [synth.SeqSpec(20, 30, 10, 17, (6, 20, 34), tail=7), synth.SeqSpec(0, 1, 1, 40, (0, 0, 0))]
    w = synth.Workload("alignment", dtype, dt16, 14, 2, hd, g, 64, 1.0, specs, 9500 + hd + g + dtype, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = np.random.default_rng(7).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    cap, off16 = H.capacities(w, slack=4)
    run = H.run_gpu(bt, cap=cap, off16=off16, splits=8, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False, cap=cap, off16=off16)
    sm, rng = 1.0 / float(np.sqrt(hd)), np.random.default_rng(8)

    moved = W.PackedKV(w.B, w.Hkv, hd, g, H.TORCH_DT[dt16], cap, off16, fill=0)
    moved.k16, moved.v16 = _off_by_one(moved.k16), _off_by_one(moved.v16)
    moved.desc.k16, moved.desc.v16 = moved.k16.data_ptr(), moved.v16.data_ptr()
    t = bt.t
    scores = torch.from_numpy(sc).cuda()
    _, perm, seg = W.wq_assign_bits(run.ctx, scores, H.i32(t.win_off), 64, W.MODE_QUOTA, H.i32(t.quota), None, w.top_bits, w.pin_first)
    W.wq_reorder_quantize(run.ctx, H.to_dev(bt.K, dtype), H.to_dev(bt.V, dtype), H.i32(t.kv_off), H.i32(t.win_size), H.i32(t.win_off), perm, seg,
                          int(t.kv_off[-1]), moved)
    for b in range(w.B):
        a, n = int(off16[b]), int(o.pk.len16[b])
        assert torch.equal(moved.k16[a:a + n], run.pk.k16[a:a + n]) and torch.equal(moved.v16[a:a + n], run.pk.v16[a:a + n])

    q = H.to_dev(bt.q, dtype)
    for cache, query in ((run.pk, _off_by_one(q)), (moved, q), (moved, _off_by_one(q))):
        for splits in (0, 1, 3):
            out = W.wq_decode_attention(run.ctx, query, cache, sm, splits, 700, W.DECODE_AUTO)
            assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, splits
    kn, vn = (synth.round_to(rng.standard_normal((w.B, 2, hd)).astype(np.float32), dt16) for _ in range(2))
    for b in range(w.B):
        r = int(o.pk.off16[b] + o.pk.len16[b])
        o.pk.k16[r], o.pk.v16[r] = kn[b], vn[b]
        o.pk.len16[b] += 1
    want = O.decode_attention(bt.q, o.pk, sm)
    for cache in (run.pk, moved):
        out = W.wq_decode_append_attention(run.ctx, q, cache, _off_by_one(H.to_dev(kn, dt16)), _off_by_one(H.to_dev(vn, dt16)), sm, 3, 700)
        assert H.attention_error(out.cpu().numpy(), want) <= TIGHT
        assert np.array_equal(cache.len16.cpu().numpy(), o.pk.len16)
    assert run.ctx.device_status() == 0
