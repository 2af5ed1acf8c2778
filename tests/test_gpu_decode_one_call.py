"""The one-call decode step against append, then attend (needs an MI355X)."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,g", [(64, 32), (64, 64)])
@pytest.mark.parametrize("seed", range(6))
def test_automatic_counts_by_length_are_those_of_the_grown_cache(hd, g, seed):
    """Uneven sequences whose 16-bit segments hold whole blocks (0 to 3 of 32 rows), so that the appended token begins a new
    block, the dearest of all: the automatic split counts by length must see it, or the one-call form cuts the sequences at other
    places than append followed by attention does.  With fixed shares both give the same bits."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    rng = np.random.default_rng(8100 + seed)
    specs = [synth.SeqSpec(60, 16, 16, 32, (10, 20, 30))]
    for b in range(int(rng.integers(2, 11))):
        n = int(rng.integers(0, 25))
        top = int(rng.integers(0, n + 1))
        specs.append(synth.SeqSpec(n, 16, 16, 32 * int(rng.integers(0 if n else 1, 4)), (top, (n - top) // 2, n - top - (n - top) // 2)))
    w = synth.Workload("one-call", synth.BF16, synth.BF16, 8, 2, hd, g, 64, 1.0, specs, 8200 + seed, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    sc = rng.standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    cap, off16 = H.capacities(w, slack=2)
    run = H.run_gpu(bt, cap=cap, off16=off16, splits=1, with_scores=False, scores_override=sc)
    ctx = W.Context(W.workspace_bytes(w.B, w.Hq, hd, 64))
    q, sm, longest = H.to_dev(bt.q, w.dtype), 0.125, 1000
    algo = W.DECODE_AUTO | W.DECODE_BY_LENGTH | W.DECODE_FIXED_SHARES
    kn, vn = (H.to_dev(synth.round_to(rng.standard_normal((w.B, 2, hd)).astype(np.float32), w.dtype), w.dtype) for _ in range(2))
    saved = run.pk.k16.clone(), run.pk.v16.clone(), run.pk.len16.clone()
    W.wq_append_kv(ctx, kn, vn, run.pk)
    two = W.wq_decode_attention(ctx, q, run.pk, sm, 0, longest, algo)
    want = run.pk.k16.clone(), run.pk.v16.clone(), run.pk.len16.clone()
    for dst, src in zip((run.pk.k16, run.pk.v16, run.pk.len16), saved):
        dst.copy_(src)
    one = W.wq_decode_append_attention(ctx, q, run.pk, kn, vn, sm, 0, longest, algo)
    for got, exp in zip((run.pk.k16, run.pk.v16, run.pk.len16), want):
        assert torch.equal(got, exp)
    assert bool((one == two).all())
    assert ctx.device_status() == 0
