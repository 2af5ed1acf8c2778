"""Scales with their sign bit set (needs an MI355X): a group of nearly equal fp32 values whose smallest one rounds up to f16 (0.3 does)
has its largest value below its stored minimum, and the quantizer stores a negative scale."""
import numpy as np
import pytest

from paper_2605_02262_amd import synth
from tests.test_gpu_decode_precision import SHAPES, _group_errors

pytestmark = pytest.mark.gpu

assert float(np.float16(0.3)) > 0.3


def _batch(hd, g, frames=40):
    specs = [synth.SeqSpec(frames, 64, 64, 21, (frames // 4, frames // 4, frames - 2 * (frames // 4))), synth.SeqSpec(7, 64, 64, 3, (0, 0, 7)), synth.SeqSpec(3, 33, 33, 40, (1, 1, 1))]
    w = synth.Workload("negative", synth.F32, synth.F16, 14, 2, hd, g, 64, 0.5, specs, 700 + hd + g, pin_first=0)
    return synth.batch(w, with_embeddings=False)


def _negative(o, want_share):
    """Share of the batch's value groups whose scale is negative, checked to be there at every width."""
    for c in range(3):
        used = int(o.pk.cls_off[c][-1])
        meta = o.pk.packed_meta(c)[1]
        s = (meta[:, :used * (o.pk.hd // o.pk.group)] & 0xFFFF).astype(np.uint16).view(np.float16)
        assert (s < 0).mean() > want_share, c


@pytest.mark.parametrize("low", [8, 12])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_places_of_one_and_four_groups(hd, g, low):
    """Values of deviation 2^-low; a token of 0.3 in 64, with a logit far below the others', so that only its scale counts.  Bounds as in test_gpu_decode_split: the vector kernel's own errors against
    64 bits.  (Placed by the bit patterns of negative scales the weights were off by up to 6e-4 of their group.)"""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    bt = _batch(hd, g)
    bt.V *= np.float32(2.0 ** -low)
    bt.V[::64] = np.float32(0.3)
    bt.q[:, :, 0], bt.K[:, :, 0], bt.K[::64, :, 0] = 16.0, 0.0, -30.0
    sc = np.random.default_rng(7).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    run = H.run_gpu(bt, splits=16, with_scores=False, scores_override=sc)
    bt.q = synth.round_to(bt.q, synth.F16)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False)
    _negative(o, 0.01)
    q, sm = H.to_dev(bt.q, synth.F16), 1.0 / float(np.sqrt(hd))
    for splits in (1, 4, 16):
        got = {a: W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2700, a).cpu().numpy() for a in (W.DECODE_AUTO, W.DECODE_GENERIC)}
        vector = _group_errors(got[W.DECODE_GENERIC], o.out, g).max()
        assert _group_errors(got[W.DECODE_AUTO], o.out, g).max() <= max(4 * vector, 2.0 ** -20), splits
        rms = {a: np.linalg.norm(x - o.out) for a, x in got.items()}
        assert rms[W.DECODE_AUTO] <= 2 * rms[W.DECODE_GENERIC], splits
    assert run.ctx.device_status() == 0


@pytest.mark.parametrize("frames", [20, 200], ids=["one launch", "three launches"])
@pytest.mark.parametrize("hd,g", [(128, 64), (64, 32)])
def test_largest_value_scale_of_two_groups(hd, g, frames):
    """A token of 0.3 in the first group of every 16th token of ordinary values, the rest of the values 2^-14 of them: a block is in the
    table by its largest scale whatever their signs, and the f16 weights are placed by that one.  (With a negative scale the largest
    bit pattern of its block, such blocks were left out and their weights overflowed.)"""
    from tests import wq_harness as H
    bt = _batch(hd, g, frames)
    n = bt.V.shape[0] // 2
    bt.V[n:] = synth.round_to(bt.V[n:] * np.float32(2.0 ** -14), synth.F16)        # (rows that stay 16-bit are compared bit for bit)
    bt.V[:n:16, :, :g] = np.float32(0.3)
    sc = np.random.default_rng(7).standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    run = H.run_gpu(bt, splits=16, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False)
    _negative(o, 0.01)
    H.assert_packed_equal(run, o)
    assert H.attention_error(run.out.cpu().numpy(), o.out) <= H.ATTN_TOL
    assert run.ctx.device_status() == 0
