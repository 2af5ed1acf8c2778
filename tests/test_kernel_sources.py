"""What the kernels' sources must not contain (CPU only)."""
import glob
import os
import re

from paper_2605_02262_amd import build


def test_no_vector_instruction_in_inline_assembly():
    """The compiler puts the wait states that a matrix instruction needs behind a vector write of its operand (two on gfx950), and
    those of the other register hazards, between instructions that it selects itself; inline assembly is opaque to it.  With
    v_fma_mixhi_f16 written that way, 60 matrix products read an operand one wait state too early."""
    statements = 0
    for path in sorted(glob.glob(os.path.join(build.CSRC, "*"))):
        text = open(path).read()
        for m in re.finditer(r"\basm\b\s*(?:volatile\s*)?\(\s*((?:\"[^\"]*\"\s*)+)", text):
            statements += 1
            assert not re.search(r"\b(v|ds|global|buffer|flat|scratch)_\w", m[1]), (os.path.basename(path), m[1])
    assert statements > 0
