"""The column kernels of the long columns (sg_colfs.o) as built: scratch (register
spills) per lane, which costs HBM traffic once for every column.  The bounds are
the figures at which these kernels were measured and kept; a change that holds
more registers across a phase shows here before it shows in a time."""
import os
import re

import pytest

from paper_1904_07400_amd import build

OBJ = os.path.join(build.HERE, "_build", "sg_colfs.o")

# pattern of the demangled-enough name -> most bytes of scratch per lane
BOUNDS = [
    # adjoint columns of 8192 in FP64: 376 with the outputs formed one by one, 484 (and
    # 1.1 to 1.18 times the time) with all of them held for the padding values' share
    (r"k_colfs_adjIddLi8192", 380),
    (r"k_colfs_adjIf", 0),
    (r"k_colw_adjIffLi4096ELi0", 0),
    (r"k_colwIffLi4096", 96),
    (r"k_colfs3", 0),
]


@pytest.mark.parametrize("pattern,limit", BOUNDS, ids=[b[0] for b in BOUNDS])
def test_scratch(pattern, limit):
    if not os.path.exists(OBJ):
        pytest.skip("no object files (build first)")
    hit = [(r[0], r[1]) for r in build.kernel_resources(OBJ) if re.search(pattern, r[0])]
    assert hit, pattern
    assert all(s <= limit for _, s in hit), hit
