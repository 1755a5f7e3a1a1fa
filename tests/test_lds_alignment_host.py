"""Dynamic LDS that kernels read and write 16 bytes at a time: every declaration has to say so.  A plain `extern __shared__ float[]`
starts right behind a kernel's static words (at byte 4 behind one int), which no 16-byte access may assume."""
import os
import re

import paper_2602_11808_amd as dfk

CSRC = os.path.join(os.path.dirname(os.path.abspath(dfk.__file__)), "csrc")


def test_every_dynamic_lds_array_is_declared_with_16_byte_alignment():
    decls = []
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".h")):
            with open(os.path.join(CSRC, name)) as f:
                decls += [(name, n, l.strip()) for n, l in enumerate(f, 1) if re.search(r"\bextern\s+__shared__", l)]
    assert len(decls) >= 10
    loose = [d for d in decls if not re.search(r"aligned\((16|32|64|128)\)", d[2])]
    assert not loose, loose
