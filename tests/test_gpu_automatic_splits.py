"""Automatic split counts (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [64, 32])
def test_the_workspace_size_does_not_change_the_bits(group):
    """One request, 20000 rows in 16 bits: the most expensive blocks, so that the launch would use more splits than the plain count
    leaves room for.  With fixed shares the bits show the count."""
    from paper_2605_02262_amd import binding as W
    B, Hkv, hd, n = 1, 2, 128, 20000
    gen = torch.Generator(device="cuda").manual_seed(5)
    cache = W.PackedKV(B, Hkv, hd, group, torch.bfloat16, [0, 0, 0], [0, n])
    cache.k16.copy_(torch.randn(n, Hkv, hd, generator=gen, device="cuda"))
    cache.v16.copy_(torch.randn(n, Hkv, hd, generator=gen, device="cuda"))
    cache.len16.fill_(n)
    q = torch.randn(B, 14, hd, generator=gen, device="cuda").to(torch.bfloat16)
    plain = W.auto_splits(B, Hkv, n)
    got = []
    for splits in (plain, 64, 256):
        ctx = W.Context(W.workspace_bytes(B, 14, hd, splits))
        got.append(W.wq_decode_attention(ctx, q, cache, 0.088, 0, n, W.DECODE_FIXED_SHARES))
        assert ctx.device_status() == 0
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])


@pytest.mark.parametrize("hd,group", [(64, 32), (128, 128)])
def test_by_length_takes_effect_where_capacities_exceed_contents(hd, group):
    """Uneven sequences in a cache of just their size, in one whose classes have room for all tokens each and whose 16-bit segment
    has room to grow, and in one with room for about as many tokens as sequences of the longest length would have: the kernel
    finds the same counts by length, hence, with fixed shares, the same bits."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    rng = np.random.default_rng(11)
    specs = [synth.SeqSpec(100, 32, 32, 40, (20, 40, 40))] + [synth.SeqSpec(n, 32, 32, 33, (n // 3, n // 3, n - 2 * (n // 3))) for n in range(2, 40, 3)]
    w = synth.Workload("roomy", synth.BF16, synth.BF16, 8, 2, hd, group, 64, 1.0, specs, 9700, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = rng.standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    total, longest = int(bt.t.kv_off[-1]), int(np.diff(bt.t.kv_off).max())
    q, ctx = H.to_dev(bt.q, w.dtype), W.Context(W.workspace_bytes(w.B, w.Hq, hd, 64))
    tight, off16 = H.capacities(w)
    got = []
    spare = w.B * longest - sum(tight) - int(off16[-1])
    for cap, off in ((tight, off16), ([total] * 3, off16 + 1500 * np.arange(w.B + 1)), (tight, off16 + spare // w.B * np.arange(w.B + 1))):
        run = H.run_gpu(bt, cap=cap, off16=off.astype(np.int32), splits=1, with_scores=False, scores_override=sc)
        got.append(W.wq_decode_attention(ctx, q, run.pk, 0.1, 0, longest, W.DECODE_BY_LENGTH | W.DECODE_FIXED_SHARES))
    even = W.wq_decode_attention(ctx, q, run.pk, 0.1, 0, longest, W.DECODE_FIXED_SHARES)
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2]) and not torch.equal(got[0], even)
    assert ctx.device_status() == 0


@pytest.mark.parametrize("B,n,group", [(1, 12800, 64), (9, 4000, 64), (1, 12800, 32), (3, 700, 128)])
def test_both_merges_take_the_same_count(B, n, group):
    """The merge inside the kernel and the second kernel's: the same bits under fixed shares, automatic counts included.  A launch
    without any merge leaves the same partials."""
    from paper_2605_02262_amd import binding as W
    Hkv, hd = 4, 128
    gen = torch.Generator(device="cuda").manual_seed(6)
    cache = W.PackedKV(B, Hkv, hd, group, torch.bfloat16, [0, 0, 0], [n * b for b in range(B + 1)])
    cache.k16.copy_(torch.randn(n * B, Hkv, hd, generator=gen, device="cuda"))
    cache.v16.copy_(torch.randn(n * B, Hkv, hd, generator=gen, device="cuda"))
    cache.len16.copy_(n - torch.arange(B, dtype=torch.int32) * 31)
    q = torch.randn(B, 28, hd, generator=gen, device="cuda").to(torch.bfloat16)
    ctx = W.Context(W.workspace_bytes(B, 28, hd, W.auto_splits(B, Hkv, n)))          # (zero)
    inside = W.wq_decode_attention(ctx, q, cache, 0.088, 0, n, W.DECODE_FIXED_SHARES)
    for flags in (W.DECODE_SEPARATE_MERGE, W.DECODE_SEPARATE_MERGE | W.DECODE_BY_LENGTH):
        partials = ctx.ws[16384:].clone()
        assert torch.equal(W.wq_decode_attention(ctx, q, cache, 0.088, 0, n, W.DECODE_FIXED_SHARES | flags), inside)
        ctx.ws[16384:].zero_()
        W.wq_decode_attention(ctx, q, cache, 0.088, 0, n, W.DECODE_FIXED_SHARES | W.DECODE_PARTIALS_ONLY)
        assert torch.equal(ctx.ws[16384:], partials)
    assert ctx.device_status() == 0


@pytest.mark.parametrize("B,n,Hkv,group", [(1, 1600, 4, 64), (8, 12800, 4, 64), (40, 3200, 4, 64), (40, 3200, 4, 128), (64, 700, 1, 64)])
def test_even_sequences_get_the_plain_count_by_length_too(B, n, Hkv, group):
    """The flag for lengths on sequences that are equally long: the count of the call without it, hence the same bits under fixed
    shares; a step in one call included."""
    from paper_2605_02262_amd import binding as W
    gen = torch.Generator(device="cuda").manual_seed(7)
    cache = W.PackedKV(B, Hkv, 128, group, torch.bfloat16, [0, 0, 0], [(n + 4) * b for b in range(B + 1)])
    cache.k16.copy_(torch.randn((n + 4) * B, Hkv, 128, generator=gen, device="cuda"))
    cache.v16.copy_(torch.randn((n + 4) * B, Hkv, 128, generator=gen, device="cuda"))
    cache.len16.fill_(n)
    q = torch.randn(B, 7 * Hkv, 128, generator=gen, device="cuda").to(torch.bfloat16)
    kn = torch.randn(B, Hkv, 128, generator=gen, device="cuda").to(torch.bfloat16)
    ctx = W.Context(W.workspace_bytes(B, 7 * Hkv, 128, W.auto_splits(B, Hkv, n + 4)))
    got = []
    for flags in (W.DECODE_FIXED_SHARES, W.DECODE_FIXED_SHARES | W.DECODE_BY_LENGTH):
        cache.len16.fill_(n)
        got.append((W.wq_decode_attention(ctx, q, cache, 0.088, 0, n + 4, flags),
                    W.wq_decode_append_attention(ctx, q, cache, kn, kn, 0.088, 0, n + 4, flags)))
        assert cache.len16.tolist() == [n + 1] * B
    for a, b in zip(*got):
        assert torch.equal(a, b)
    assert ctx.device_status() == 0
