"""Decode with one and four groups per head where the weights' two f16 values, their place and the codes' offsets could go wrong
(needs an MI355X).  Bounds as in test_gpu_decode_precision: the vector kernel's own errors against 64 bits."""
import numpy as np
import pytest

from paper_2605_02262_amd import synth
from tests.test_gpu_decode_precision import SHAPES, _group_errors

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", ["rising", "falling", "far groups", "tiny", "large", "outlier last", "keys off zero", "constant", "far queries"])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_places_and_offsets(hd, g, shape):
    """Value scales that grow and shrink along the walk by 2^16, groups 2^10 apart, f16's smallest and largest magnitudes, one
    large token at the end of the stream; keys whose groups do not straddle zero; groups of equal entries (scale 1); half of a head's
    query 2^-10 of the other half, its keys 2^10 times as large."""
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = [synth.SeqSpec(40, 64, 64, 21, (10, 15, 15)), synth.SeqSpec(7, 64, 64, 3, (0, 0, 7)), synth.SeqSpec(3, 33, 33, 40, (1, 1, 1))]
    w = synth.Workload("split", synth.F16, synth.F16, 14, 2, hd, g, 64, 0.5, specs, 4000 + hd + g, pin_first=0)
    bt = synth.batch(w, with_embeddings=False)
    n = bt.V.shape[0]
    at = np.linspace(0.0, 1.0, n)[:, None, None]
    if shape == "rising":
        bt.V *= 2.0 ** (np.round(16 * at) - 8)
    elif shape == "falling":
        bt.V *= 2.0 ** (8 - np.round(16 * at))
    elif shape == "far groups":
        bt.V *= np.repeat(2.0 ** (4 - 10.0 * (np.arange(hd // g) % 2)), g)
    elif shape == "tiny":
        bt.V *= 2.0 ** -12
    elif shape == "large":
        bt.V *= 2.0 ** 13
    elif shape == "outlier last":
        bt.V[bt.t.kv_off[1] - 30] *= 2.0 ** 10
    elif shape == "keys off zero":
        bt.K[:, 0] = np.abs(bt.K[:, 0]) + 3.0
        bt.K[:, 1] = -np.abs(bt.K[:, 1]) - 3.0
    elif shape == "far queries":
        bt.q[:, :, hd // 2:] *= 2.0 ** -10
        bt.K[:, :, hd // 2:] *= 2.0 ** 10
    else:
        bt.K[::3] = 0.25
        bt.V[1::3] = -0.5
    for name in ("K", "V", "q"):
        setattr(bt, name, synth.round_to(getattr(bt, name).astype(np.float32), w.dtype))
    rng = np.random.default_rng(7)
    sc = rng.standard_normal(int(bt.t.win_off[-1])).astype(np.float32)
    run = H.run_gpu(bt, splits=16, with_scores=False, scores_override=sc)
    o = H.run_oracle(bt, scores_override=sc, with_scores=False)
    q, sm = H.to_dev(bt.q, w.dtype), 1.0 / float(np.sqrt(hd))
    for splits in (1, 4, 16):
        got = {a: W.wq_decode_attention(run.ctx, q, run.pk, sm, splits, 2700, a).cpu().numpy() for a in (W.DECODE_AUTO, W.DECODE_GENERIC)}
        vector = _group_errors(got[W.DECODE_GENERIC], o.out, g).max()
        assert _group_errors(got[W.DECODE_AUTO], o.out, g).max() <= max(4 * vector, 2.0 ** -20), splits
        rms = {a: np.linalg.norm(x - o.out) for a, x in got.items()}
        assert rms[W.DECODE_AUTO] <= 2 * rms[W.DECODE_GENERIC], splits
    assert run.ctx.device_status() == 0


@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16])
@pytest.mark.parametrize("hd,g", SHAPES)
def test_softmax_scales_of_any_size(hd, g, dtype):
    """Softmax scales from fp32's smallest to its largest number, with queries of zeros and of the type's smallest and largest magnitudes:
    the power of two that brings a query into f16, times the softmax scale, can lie outside fp32's range.  Logits that are zero, or
    nothing beside one, weigh all tokens alike, those past a class's end (every class here has a partial block) not at all.  2^-18: fp32
    sums of 300 terms that cancel to a tenth."""
    from oracle import wq_oracle as O
    from paper_2605_02262_amd import binding as W
    from tests import wq_harness as H
    specs = [synth.SeqSpec(9, 33, 33, 5, (3, 3, 3)), synth.SeqSpec(3, 17, 17, 40, (1, 1, 1))]
    w = synth.Workload("scale", dtype, dtype, 14, 2, hd, g, 64, 0.5, specs, 100 + hd + g, pin_first=0)
    sc = np.random.default_rng(1).standard_normal(18).astype(np.float32)
    small, large = (2.0 ** -126, 2.0 ** 120) if dtype == synth.BF16 else (2.0 ** -24, 2.0 ** 14)
    for sm, q_to, k_to in ((2.0 ** -126, 0.0, 1.0), (2.0 ** -60, 0.0, 1.0), (2.0 ** -60, small, 1.0), (2.0 ** 100, 0.0, 1.0), (2.0 ** 126, large, 0.0)):
        bt = synth.batch(w, with_embeddings=False)
        bt.q = np.sign(bt.q) * np.float32(q_to)
        bt.K *= np.float32(k_to)
        run = H.run_gpu(bt, splits=4, with_scores=False, scores_override=sc)
        want = O.decode_attention(np.zeros_like(bt.q), H.run_oracle(bt, scores_override=sc, with_scores=False).pk, 1.0)      # (equal logits)
        q = H.to_dev(bt.q, dtype)
        for algo in (W.DECODE_AUTO, W.DECODE_GENERIC):
            got = W.wq_decode_attention(run.ctx, q, run.pk, sm, 4, 400, algo).cpu().numpy()
            assert np.isfinite(got).all(), (sm, q_to, algo)
            assert _group_errors(got, want, g).max() <= 2.0 ** -18, (sm, q_to, algo)
