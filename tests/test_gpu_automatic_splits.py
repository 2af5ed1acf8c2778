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
