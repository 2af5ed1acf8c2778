"""Decode attention with one and four groups per head where 16 bits anywhere would show (needs an MI355X).

The matrix-core kernel has the vector kernel's accuracy here (WQ_DECODE_GENERIC, fp32 throughout) by other operations: products of f16
numbers that hold codes, queries and weights to 23 bits or more, scales and offsets after the contraction, fp32 sums."""
import numpy as np
import pytest
import torch

from paper_2605_02262_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [(128, 32), (128, 128), (64, 64)]


def _group_errors(got, want, group):
    """Largest error of every group of every head, relative to that group's own largest entry."""
    B, Hq, hd = want.shape
    d = np.abs(got.astype(np.float64) - want).reshape(B, Hq, hd // group, group).max(-1)
    s = np.abs(want).reshape(B, Hq, hd // group, group).max(-1)
    return d / np.where(s > 0, s, 1.0)


def _caches(hd, g, dtype, spread, Hkv=2, rep=7, seed=0):
    from tests import wq_harness as H
    specs = [synth.SeqSpec(32, 64, 64, 77, (8, 12, 12)), synth.SeqSpec(9, 64, 64, 33, (0, 0, 9)), synth.SeqSpec(5, 64, 64, 9, (1, 2, 2))]
    w = synth.Workload("precision", dtype, dtype, rep * Hkv, Hkv, hd, g, 64, 1.0, specs, 9000 + hd + g + dtype + seed, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    rng = np.random.default_rng(seed)
    if spread == "heads":              # one KV head's values 2^12 smaller than the other's
        bt.V[:, 1] *= 2.0 ** -12
    elif spread == "groups":           # a head's groups 2^4 apart from one another
        bt.V *= np.repeat(2.0 ** -(4.0 * np.arange(hd // g)), g).astype(np.float32)
    elif spread == "tokens":           # values of a token up to 2^12 smaller than another's
        bt.V *= (2.0 ** -rng.integers(0, 13, size=(bt.V.shape[0], 1, 1))).astype(np.float32)
    elif spread == "query":            # query channels up to 2^14 apart, the keys half of that the other way; logits of deviation 2
        e = rng.integers(-14, 1, size=hd)
        bt.q *= (2.0 ** e).astype(np.float32)
        bt.K *= (2.0 ** -(e // 2)).astype(np.float32)
        kg = bt.K.reshape(-1, Hkv, hd // g, g)
        step = (kg.max(-1) - kg.min(-1)) / 3                            # of 2-bit codes: a key is off by up to half of it
        var = (kg ** 2 + step[..., None] ** 2 / 12).reshape(-1, Hkv, hd).mean(0)
        dev = np.sqrt((bt.q.reshape(w.B, Hkv, rep, hd) ** 2 * var[None, :, None]).sum(-1) / hd).reshape(w.B, Hkv * rep, 1)
        bt.q *= (2.0 / dev).astype(np.float32)
    elif spread == "large logits":
        bt.q *= 16
    for n in ("K", "V", "q"):
        setattr(bt, n, synth.round_to(getattr(bt, n), dtype))
    sc = rng.standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    run = H.run_gpu(bt, splits=16, with_scores=False, scores_override=sc)
    return w, bt, run, H.run_oracle(bt, scores_override=sc, with_scores=False)


@pytest.mark.parametrize("spread", ["none", "heads", "groups", "tokens", "query", "large logits"])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_no_less_precise_than_the_vector_kernel(hd, g, dtype, spread):
    """Errors against 64 bits of every group by its own magnitude.  Bound: what the vector kernel shows on the same input, four
    times that (the largest of a few hundred rounding errors moves by such a factor when sums are ordered differently), and
    2^-20 where it happens to show next to nothing (a softmax over few tokens).  Weights in two f16 values placed by the
    largest value scale were 20 to 100 times off here."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    w, bt, run, o = _caches(hd, g, dtype, spread)
    q, sm = H.to_dev(bt.q, dtype), 1.0 / float(np.sqrt(hd))
    for splits in (1, 5, 16):
        got = {a: W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, a).cpu().numpy() for a in (W.DECODE_AUTO, W.DECODE_GENERIC)}
        vector = _group_errors(got[W.DECODE_GENERIC], o.out, g).max()
        assert _group_errors(got[W.DECODE_AUTO], o.out, g).max() <= max(4 * vector, 2.0 ** -20), splits
        # (and as a whole: root mean square over all outputs)
        rms = {a: np.linalg.norm(x - o.out) for a, x in got.items()}
        assert rms[W.DECODE_AUTO] <= 2 * rms[W.DECODE_GENERIC], splits


@pytest.mark.parametrize("hd,g", SHAPES)
def test_value_scale_table_is_not_read_and_bits_repeat(hd, g):
    """v_scale_max belongs to the f16 weights of two groups; without any flag a split count fixes every bit."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    w, bt, run, o = _caches(hd, g, synth.BF16, "none")
    q, sm = H.to_dev(bt.q, w.dtype), 1.0 / float(np.sqrt(hd))
    for splits, flags in ((1, 0), (5, 0), (16, 0), (16, W.DECODE_BY_LENGTH)):
        first = W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, flags)
        for fill in (0.0, float("nan"), 3e38):
            run.pk.v_scale_max.fill_(fill)
            assert torch.equal(W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, flags), first), (splits, fill)
        assert torch.equal(W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, flags | W.DECODE_FIXED_SHARES), first)
        assert torch.equal(W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, flags | W.DECODE_SEPARATE_MERGE), first) or flags


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_query_of_the_other_16_bit_type(hd, g, dtype):
    """An fp16 query on a bf16 cache (the 16-bit rows are then the vector kernel's) and the other way round."""
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    from tests.test_gpu_decode_groups import TIGHT
    w, bt, run, o = _caches(hd, g, dtype, "none")
    other = synth.F16 if dtype == synth.BF16 else synth.BF16
    qv = synth.round_to(bt.q, other)
    q, sm = H.to_dev(qv, other), 1.0 / float(np.sqrt(hd))
    want = O.decode_attention(qv, o.pk, sm)
    for splits in (1, 5):
        out = W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2200, W.DECODE_AUTO)
        assert H.attention_error(out.cpu().numpy(), want) <= TIGHT, splits
    assert run.ctx.device_status() == 0


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_infinities_in_16_bit_rows(hd, g, dtype):
    """A key entry that makes a logit -inf leaves its token out; an infinite value entry (in the last row, too, which ends a
    partial block) makes its channel infinite and no other.  As the vector kernel has it."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    w, bt, run, o = _caches(hd, g, dtype, "none", rep=1)
    q, sm = H.to_dev(bt.q, dtype), 1.0 / float(np.sqrt(hd))
    off16, len16 = run.pk.off16.cpu().numpy(), run.pk.len16.cpu().numpy()
    clean = W.wq_decode_attention(run.ctx, q, run.pk, sm, 3, 2200, W.DECODE_AUTO)
    for b, row in ((0, 3), (1, 32), (2, 0)):                            # keys: -inf logits for both heads
        for h in range(2):
            ch = 5 + h
            run.pk.k16[off16[b] + row, h, ch] = -float("inf") if float(q[b, h, ch]) > 0 else float("inf")
    got = [W.wq_decode_attention(run.ctx, q, run.pk, sm, 3, 2200, a) for a in (W.DECODE_AUTO, W.DECODE_GENERIC)]
    assert bool(torch.isfinite(got[0]).all()) and bool(torch.isfinite(got[1]).all()) and not torch.equal(got[0], clean)
    assert float((got[0] - got[1]).abs().max()) <= 2.0 ** -17 * float(got[1].abs().max())
    for b in range(w.B):
        run.pk.v16[off16[b] + len16[b] - 1, 0, 7] = float("inf")        # the last row
        run.pk.v16[off16[b], 1, hd - 1] = -float("inf")
    got = [W.wq_decode_attention(run.ctx, q, run.pk, sm, 3, 2200, a) for a in (W.DECODE_AUTO, W.DECODE_GENERIC)]
    at = torch.isinf(got[1])
    assert int(at.sum()) >= w.B                                         # (-inf rows of the keys may have left a -inf value out)
    assert torch.equal(torch.isnan(got[0]), torch.isnan(got[1])) and torch.equal(torch.isinf(got[0]), at)
    assert torch.equal(got[0][at], got[1][at])
