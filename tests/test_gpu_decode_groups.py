"""Decode attention with one and four groups per head on the matrix cores, against the oracle (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth

pytestmark = pytest.mark.gpu

# With 16-bit queries these group counts have the errors of fp32 arithmetic.  Relative to a vector's largest entry: a logit of
# up to 2^5 is rounded to 2^-19 in a sum of up to 128 products (a few such roundings at random signs, 2^-17 or so), which
# its weight takes on relatively; the hardware's exponential is good to 2^-21 or so of the weight, sums of positive weights
# to a few 2^-22.  Together about 2^-17; 2^-15 leaves a factor of four, and is 60 times tighter than the bound of one f16
# weight.  (test_gpu_decode_precision compares with the vector kernel's own error, group by group.)
TIGHT = 2.0 ** -15


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
@pytest.mark.parametrize("hd,g", [(128, 32), (128, 128), (64, 64)])
def test_one_and_four_groups_keep_fp32_accuracy(hd, g, dtype):
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    # class lengths around the 16-token tile and the 32-token block (1, 15, 16, 17, 31, 32, 33), one class alone, none at all
    specs = [synth.SeqSpec(49, 1, 1, 31, (1, 15, 33)), synth.SeqSpec(65, 1, 1, 0, (16, 17, 32)), synth.SeqSpec(31, 1, 1, 33, (31, 0, 0)),
             synth.SeqSpec(0, 1, 1, 1, (0, 0, 0)), synth.SeqSpec(40, 30, 10, 17, (20, 50, 50), tail=7)]
    w = synth.Workload("groups", dtype, dtype, 7 * 2, 2, hd, g, 64, 1.0, specs, 31 + hd + g + dtype, pin_first=0)
    bt = synth.batch(w)
    cap, off16 = H.capacities(w, slack=2)
    run = H.run_gpu(bt, cap=cap, off16=off16, splits=65)
    o = H.run_oracle(bt, scores_override=run.scores.cpu().numpy(), cap=cap, off16=off16)
    H.assert_packed_equal(run, o)
    q, sm = H.to_dev(bt.q, dtype), 1.0 / float(np.sqrt(hd))
    for splits, flags in ((1, 0), (1, W.DECODE_FIXED_SHARES), (3, 0), (64, 0), (65, 0), (3, W.DECODE_SEPARATE_MERGE), (8, W.DECODE_BY_LENGTH)):
        lse = torch.empty(w.B, w.Hq, device="cuda")
        out = W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 1300, flags, lse=lse)
        err = H.attention_error(out.cpu().numpy(), o.out)
        assert err <= TIGHT, (splits, flags)
        assert np.abs(lse.cpu().numpy() - o.lse).max() <= 1e-4          # a sum of weights accurate to 2^-15
    rng = np.random.default_rng(3)
    for step in range(2):                                               # two appended tokens, one launch each
        kn, vn = (synth.round_to(rng.standard_normal((w.B, w.Hkv, hd)).astype(np.float32), dtype) for _ in range(2))
        out = W.wq_decode_append_attention(run.ctx, q, run.pk, H.to_dev(kn, dtype), H.to_dev(vn, dtype), sm, 3, 1300, W.DECODE_AUTO)
        for b in range(w.B):
            r = int(o.pk.off16[b] + o.pk.len16[b])
            o.pk.k16[r], o.pk.v16[r] = kn[b], vn[b]
            o.pk.len16[b] += 1
        err = H.attention_error(out.cpu().numpy(), O.decode_attention(bt.q, o.pk, sm))
        assert err <= TIGHT, step
    assert run.ctx.device_status() == 0
