"""Dynamic LDS that is read sixteen bytes at a time says so in its declaration:
its start follows the kernel's static arrays, and without the alignment one of
them changing by a word would misalign every operand read."""

import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2304_01660_amd", "csrc")


def test_half_precision_dynamic_lds_is_sixteen_byte_aligned():
    found = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        for line in re.findall(r"extern __shared__[^;]*;", open(path).read()):
            if "_Float16" in line:
                found += 1
                assert "__align__(16)" in line, (os.path.basename(path), line)
    assert found
