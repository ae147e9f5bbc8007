"""Wait states inside inline assembly.  The compiler's hazard pass does not look
into an assembly statement, so the statement has to carry its own."""
import glob
import os
import re

import paper_2609_32420_amd as P

CSRC = os.path.join(os.path.dirname(P.__file__), "csrc")


def _statements():
    """(file, instructions) of every inline assembly statement."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        with open(path) as f:
            text = f.read()
        for m in re.finditer(r"\basm\b(?:\s+volatile)?\s*\(((?:\s*\"(?:[^\"\\]|\\.)*\")+)", text):
            body = "".join(re.findall(r"\"((?:[^\"\\]|\\.)*)\"", m.group(1)))
            yield os.path.basename(path), [x.strip() for x in re.split(r"\\n|\\t|;", body) if x.strip()]


# A scalar write of M0 needs one wait state before an instruction that takes its
# LDS address from M0.
def test_direct_loads_wait_for_m0():
    seen = 0
    for name, ins in _statements():
        for i, x in enumerate(ins):
            if not re.match(r"(global|buffer|scratch)_load_lds", x):
                continue
            seen += 1
            assert i >= 2, (name, ins)
            assert re.match(r"s_mov_b32\s+m0\b", ins[i - 2]) and ins[i - 1].startswith("s_nop"), (name, ins)
    assert seen >= 2  # the attention's and the exact mass's
