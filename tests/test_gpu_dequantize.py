"""wq_dequantize against m + s*code, bit for bit (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth
from tests.test_gpu_parity import _custom, _dense_expected

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,g", [(128, 32), (128, 64), (128, 128), (64, 32), (64, 64)])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
def test_every_value_is_rounded_once(hd, g, dtype):
    """Class lengths around the 32-token block, classes without tokens, a tail, 16-bit rows that fill no group of rows, class
    capacities beyond what is used.  m + s*code fits fp64, so rounding it to fp32 gives the fused multiply-add's value."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = [synth.SeqSpec(97, 1, 1, 31, (31, 33, 33)), synth.SeqSpec(9, 21, 21, 13, (2, 3, 4)), synth.SeqSpec(0, 10, 4, 5, (0, 0, 0)),
             synth.SeqSpec(64, 1, 1, 1, (0, 64, 0)), synth.SeqSpec(6, 32, 32, 0, (2, 2, 2), tail=7), synth.SeqSpec(32, 1, 1, 8, (32, 0, 0))]
    bt = _custom(900 + hd + g + dtype, hd, g, 3, 2, dtype, specs, pin=0)
    w = bt.w
    cap, off16 = H.capacities(w, slack=3)
    cap = [c + 32 * k for c, k in zip(cap, (5, 1, 40))]
    run = H.run_gpu(bt, cap=cap, off16=off16)
    o = H.run_oracle(bt, scores_override=run.scores.cpu().numpy(), cap=cap, off16=off16)
    H.assert_packed_equal(run, o)
    Ks, Vs = _dense_expected(o, w.dtype16)
    off = np.concatenate([[0], np.cumsum([len(k) + b % 3 for b, k in enumerate(Ks)])]).astype(np.int32)
    dense = W.PackedKV(w.B, w.Hkv, hd, g, run.pk.dtype16, [0, 0, 0], off, fill=0xA5)
    for got in (dense.k16, dense.v16):
        got.fill_(7.0)
    W.wq_dequantize(run.ctx, run.pk, dense)
    assert run.ctx.device_status() == 0
    assert dense.len16.cpu().tolist() == [len(k) for k in Ks]
    for b in range(w.B):
        a, n = int(off[b]), len(Ks[b])
        for got, want in ((dense.k16, Ks[b]), (dense.v16, Vs[b])):
            want = torch.from_numpy(want.astype(np.float32)).to(got.dtype)
            assert torch.equal(got[a:a + n].cpu().view(torch.int16), want.view(torch.int16)), b
            assert bool((got[a + n:int(off[b + 1])] == 7.0).all()), b


def test_blocks_stay_within_the_capacities():
    """A cache whose last offsets say more than the classes have room for: every block is still looked for inside its class, and
    what lies past a sequence's length is left out, so the result is that of the right offsets."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    bt = _custom(977, 128, 64, 3, 2, synth.BF16, [synth.SeqSpec(40, 16, 16, 9, (10, 14, 16)), synth.SeqSpec(9, 21, 21, 13, (2, 3, 4))], pin=0)
    run = H.run_gpu(bt)
    rows = [0] + np.cumsum(np.diff(bt.t.kv_off)).tolist()
    got = []
    for beyond in (0, 1 << 20):
        for c in range(3):
            run.pk.cls_off[c][-1] = (beyond + run.pk.cap[c]) if beyond else run.pk.cls_off[c][-1]
        dense = W.PackedKV(bt.w.B, bt.w.Hkv, 128, 64, run.pk.dtype16, [0, 0, 0], rows)
        W.wq_dequantize(run.ctx, run.pk, dense)
        got.append(dense)
    assert run.ctx.device_status() == 0
    assert got[0].k16.abs().sum() > 0 and torch.equal(got[0].k16, got[1].k16) and torch.equal(got[0].v16, got[1].v16)
    assert torch.equal(got[0].len16, got[1].len16)


def test_class_room_beyond_a_grid_dimension():
    """Room for 2^26 tokens of 8 KV heads (21 GB, hardly any of it in use): one workgroup each per block and head is more than
    one dimension of a launch takes.  The rows are those of the same cache in buffers of its size."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    bt = _custom(983, 64, 64, 8, 1, synth.BF16, [synth.SeqSpec(40, 16, 16, 9, (10, 14, 16)), synth.SeqSpec(9, 21, 21, 13, (2, 3, 4))], pin=0)
    w = bt.w
    cap, off16 = H.capacities(w)
    rows = [0] + np.cumsum(np.diff(bt.t.kv_off)).tolist()
    sc = np.random.default_rng(5).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    got = []
    for room in (cap[0], 1 << 26):
        run = H.run_gpu(bt, cap=[room, cap[1], cap[2]], off16=off16, splits=2, with_scores=False, scores_override=sc)
        dense = W.PackedKV(w.B, w.Hkv, 64, 64, run.pk.dtype16, [0, 0, 0], rows)
        W.wq_dequantize(run.ctx, run.pk, dense)
        assert run.ctx.device_status() == 0
        got.append(dense)
        del run
    assert got[0].len16.cpu().tolist() == np.diff(rows).tolist() and got[0].k16.abs().sum() > 0
    for name in ("k16", "v16", "len16"):
        assert torch.equal(getattr(got[0], name), getattr(got[1], name)), name
