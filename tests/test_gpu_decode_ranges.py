"""Decode attention where a workgroup has few blocks, and where the arrival counters change their spacing (needs an MI355X).

One group per head: the kernel then computes in fp32 (2^-15 of a vector's largest entry, see test_gpu_decode_groups), so a
block that is left out, taken twice or merged too early shows."""
import numpy as np
import pytest
import torch

from oracle import wq_oracle as O
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


@pytest.mark.parametrize("hd,g", [(64, 64), (128, 32), (128, 128)])
@pytest.mark.parametrize("rows16", [0, 1, 2, 3, 7, 17, 40])
def test_shares_of_ranges_with_blocks_in_16_bits(hd, g, rows16):
    """One and four groups per head: 1 to 65 quantized blocks beside `rows16` blocks of 16-bit rows, cut into 1 to 9 ranges whose wavefronts get
    equal shares or 5 : 3 by what their blocks cost; a larger batch whose ranges are all 5 : 3."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = []
    for n in (1, 4, 9, 16, 24, 37, 65) if rows16 < 40 else (70, 200):
        top = n // 3
        specs.append(synth.SeqSpec(n, 32, 32, max(1, 32 * rows16 - 3), (top, (n - top) // 2, n - top - (n - top) // 2)))
    w = synth.Workload("shares", synth.BF16, synth.BF16, 6, 2, hd, g, 64, 1.0, specs, 800 + rows16 + g, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = np.random.default_rng(4).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    run = H.run_gpu(bt, splits=1, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False)
    ctx = W.Context(W.workspace_bytes(w.B, w.Hq, w.hd, 9))
    q, sm = H.to_dev(bt.q, w.dtype), w.hd ** -0.5
    o.out = O.decode_attention(bt.q, o.pk, sm)
    for splits in range(1, 10):
        out = W.wq_decode_attention(ctx, q, run.pk, sm, splits, 8000)
        assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, splits
    assert ctx.device_status() == 0


@pytest.mark.parametrize("B", [14, 15, 28, 29, 50, 51, 84, 85, 126, 127])
def test_arrival_counters_at_every_spacing(B):
    """Two KV heads: a unit has 8, 4, 2 or 1 cache lines of counters up to 14, 28, 50 and 84 sequences; from 85 on the append
    counters do not fit the header, from 127 on the merge is a launch of its own.  Up to 64 splits of a few blocks."""
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = [synth.SeqSpec(3, 16, 16, 3 + b % 40, (1, 1, 1)) for b in range(B)]
    w = synth.Workload("counters", synth.BF16, synth.BF16, 16, 2, 64, 64, 64, 1.0, specs, 600 + B, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = np.random.default_rng(2).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    cap, off16 = H.capacities(w, slack=4)
    run = H.run_gpu(bt, cap=cap, off16=off16, splits=1, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False, cap=cap, off16=off16)
    ctx = W.Context(W.workspace_bytes(B, w.Hq, w.hd, 64))
    q, sm = H.to_dev(bt.q, w.dtype), 0.125
    rng = np.random.default_rng(3)
    for splits in (2, 17, 33, 64):
        out = W.wq_decode_attention(ctx, q, run.pk, sm, splits, 100)
        assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, splits
        kn, vn = (synth.round_to(rng.standard_normal((B, 2, 64)).astype(np.float32), w.dtype) for _ in range(2))
        out = W.wq_decode_append_attention(ctx, q, run.pk, H.to_dev(kn, w.dtype), H.to_dev(vn, w.dtype), sm, splits, 100)
        for b in range(B):
            r = int(o.pk.off16[b] + o.pk.len16[b])
            o.pk.k16[r], o.pk.v16[r] = kn[b], vn[b]
            o.pk.len16[b] += 1
        o.out = O.decode_attention(bt.q, o.pk, sm)
        assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, splits
        assert np.array_equal(run.pk.len16.cpu().numpy(), o.pk.len16)
    assert ctx.device_status() == 0 and int(ctx.ws[:16384].count_nonzero()) == 0        # every counter is back at zero


@pytest.mark.parametrize("B,Hkv", [(1, 2), (2, 1), (7, 3), (33, 4), (42, 3), (64, 2), (65, 2)])
def test_splits_by_length(B, Hkv):
    """Lengths from one token to 40 blocks.  Given counts and automatic ones, the latter also with a workspace for the plain
    count only; appended tokens, among them some that begin a new block.  Up to 64 sequences the kernel numbers the
    workgroups with work without gaps, beyond them a sequence's surplus workgroups return."""
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    rng = np.random.default_rng(B)
    specs = [synth.SeqSpec(40, 30, 30, 31, (8, 12, 20))]
    for b in range(1, B):
        n = int(rng.integers(0, 12)) if b % 5 else 0
        top = int(rng.integers(0, n + 1))
        specs.append(synth.SeqSpec(n, 16, 16, [1, 30, 31, 32][b % 4], (top, (n - top) // 2, n - top - (n - top) // 2)))
    w = synth.Workload("by-length", synth.BF16, synth.BF16, 3 * Hkv, Hkv, 64, 64, 64, 1.0, specs, 700 + B, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = rng.standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    cap, off16 = H.capacities(w, slack=12)
    run = H.run_gpu(bt, cap=cap, off16=off16, splits=1, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False, cap=cap, off16=off16)
    q, sm, longest = H.to_dev(bt.q, w.dtype), 0.125, 1240
    large = W.Context(W.workspace_bytes(B, w.Hq, 64, 64))
    plain = W.Context(W.workspace_bytes(B, w.Hq, 64, W.auto_splits(B, Hkv, longest)))
    for ctx, splits, flags in ((large, 0, 0), (large, 0, 0), (plain, 0, 0), (large, 0, W.DECODE_FIXED_SHARES), (large, 1, 0), (large, 5, 0), (large, 64, 0)):
        out = W.wq_decode_attention(ctx, q, run.pk, sm, splits, longest, W.DECODE_BY_LENGTH | flags)
        assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, (splits, flags)
        kn, vn = (synth.round_to(rng.standard_normal((B, Hkv, 64)).astype(np.float32), w.dtype) for _ in range(2))
        out = W.wq_decode_append_attention(ctx, q, run.pk, H.to_dev(kn, w.dtype), H.to_dev(vn, w.dtype), sm, splits, longest, W.DECODE_BY_LENGTH | flags)
        for b in range(B):
            r = int(o.pk.off16[b] + o.pk.len16[b])
            o.pk.k16[r], o.pk.v16[r] = kn[b], vn[b]
            o.pk.len16[b] += 1
        o.out = O.decode_attention(bt.q, o.pk, sm)
        assert H.attention_error(out.cpu().numpy(), o.out) <= TIGHT, (splits, flags)
        assert np.array_equal(run.pk.len16.cpu().numpy(), o.pk.len16)
    for ctx in (large, plain):
        assert ctx.device_status() == 0 and int(ctx.ws[:16384].count_nonzero()) == 0
