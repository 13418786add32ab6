"""Every device pointer of the kernels' common argument block is used by some
kernel: what none uses is workspace that the caller allocates and scalar
registers that every launch loads, for nothing."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1907_00080_amd", "csrc")


def test_every_pointer_of_the_argument_block_is_used():
    text = open(os.path.join(CSRC, "lbib_dev.h")).read()
    body = re.search(r"struct Ptrs \{(.*?)\n\};", text, re.S).group(1)
    body = re.sub(r"//[^\n]*", "", body)
    names = [n for decl in body.split(";") if "*" in decl for n in re.findall(r"\*\s*(\w+)", decl)]
    assert len(names) > 40
    kernels = "".join(open(f).read() for f in glob.glob(os.path.join(CSRC, "k_*.hip")) + [os.path.join(CSRC, "mls.h")])
    kernels = re.sub(r"//[^\n]*", "", kernels)
    unused = [n for n in names if not re.search(rf"\.{n}\b", kernels)]
    assert unused == [], unused
