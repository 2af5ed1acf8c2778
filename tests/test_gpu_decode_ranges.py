"""Decode attention where a workgroup has few blocks (needs an MI355X).

One group per head: the kernel then keeps fp32 accuracy (2^-15 of a vector's largest entry, see test_gpu_decode_groups), so a
block that is left out, taken twice or merged too early shows."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth
from tests.test_gpu_decode_groups import TIGHT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first_class", [0, 1, 2, 3])
def test_ranges_of_few_blocks(first_class):
    """1 to 41 blocks for one workgroup of eight wavefronts (one, two, three or four fixed blocks per wavefront, then drawn
    ones), most of them in one class; every launch hands the blocks out anew."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = []
    for n in (1, 2, 7, 8, 9, 15, 16, 17, 23, 24, 25, 31, 32, 33, 34, 41):
        part = max(0, n - 1)
        mix = {0: (0, 0, part), 1: (0, part, 0), 2: (part, 0, 0), 3: (0, 0, 0)}[first_class]
        specs.append(synth.SeqSpec(sum(mix), 32, 32, 5 if first_class < 3 else 32 * part + 5, mix))
    w = synth.Workload("few", synth.BF16, synth.BF16, 6, 2, 64, 64, 64, 1.0, specs, 500 + first_class, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = np.random.default_rng(1).standard_normal(max(1, int(bt.t.win_off[-1]))).astype(np.float32)[:int(bt.t.win_off[-1])]
    run = H.run_gpu(bt, splits=1, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False)
    ctx = W.Context(W.workspace_bytes(w.B, w.Hq, w.hd, 5))
    q, sm = H.to_dev(bt.q, w.dtype), 0.125
    for splits in (1, 1, 1, 2, 5):
        for flags in (0, W.DECODE_FIXED_SHARES):
            out = W.wq_decode_attention(ctx, q, run.pk, sm, splits, 1400, flags)
            assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, (splits, flags)
    assert ctx.device_status() == 0
