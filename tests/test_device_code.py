"""What the device code says of itself (no GPU needed): hand-written instructions declare what they change."""
import glob
import os
import re

import paper_2412_02252_amd as pod

CSRC = os.path.join(os.path.dirname(os.path.abspath(pod.__file__)), "csrc")


def test_instructions_that_write_m0_say_so():
    """M0 is the compiler's to use between two statements: one that changes it names it among what it clobbers."""
    seen = 0
    for f in glob.glob(os.path.join(CSRC, "*")):
        for stmt in re.findall(r"\basm\s*(?:volatile)?\s*\((.*?)\)\s*;", open(f).read(), re.S):
            if re.search(r"\b[sv]_\w+\s+m0\b", stmt):
                seen += 1
                clobbers = stmt.split(":")[-1]
                assert '"m0"' in clobbers, (os.path.basename(f), stmt)
    assert seen
