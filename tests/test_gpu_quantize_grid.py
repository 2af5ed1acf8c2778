"""The quantizer's grid: capacities far beyond use, and 16-bit rows in groups (needs an MI355X)."""
import numpy as np
import pytest

from paper_2605_02262_amd import synth
from tests.test_gpu_parity import _check, _custom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("room", [0, 64])
@pytest.mark.parametrize("dtype", [synth.BF16, synth.F16, synth.F32])
@pytest.mark.parametrize("Hkv", [1, 3])
def test_capacities_and_groups_of_rows(Hkv, dtype, room):
    """Capacities that just fit (blocks numbered by capacity) and that hold more than all rows fill (numbered by use), with every
    class empty in some sequence; 1, 7, 8 and 9 rows of 16 bits at the end of a sequence, windows among them (top tier of 16 bits)."""
    from tests import wq_harness as H
    for top_bits in (8, 16):
        specs = [synth.SeqSpec(9, 21, 21, 8, (2, 3, 4)), synth.SeqSpec(3, 16, 16, 1, (0, 1, 2)), synth.SeqSpec(0, 10, 4, 7, (0, 0, 0)),
                 synth.SeqSpec(4, 33, 33, 9, (4, 0, 0), tail=2), synth.SeqSpec(2, 32, 32, 0, (0, 0, 2))]
        bt = _custom(40 + Hkv + dtype + top_bits, 64, 32, Hkv, 2, dtype, specs, top_bits=top_bits, pin=0)
        cap, off16 = H.capacities(bt.w, slack=2)
        g, _, _ = _check(bt, H, cap=[c + 32 * room * (k + 1) for k, c in enumerate(cap)], off16=off16, splits=2)
        assert g.ctx.device_status() == 0
