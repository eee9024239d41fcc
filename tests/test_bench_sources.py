"""The benchmark ties a committed counter profile to the build by a hash of the
kernel sources: every file that the device code includes has to be in it."""
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1904_07400_amd", "csrc")


def _reached(name, seen):
    if name in seen or not os.path.exists(os.path.join(CSRC, name)):
        return
    seen.add(name)
    for inc in re.findall(r'#include "([^"]+)"', open(os.path.join(CSRC, name)).read()):
        _reached(inc, seen)


def test_hash_covers_every_kernel_source():
    sys.path.insert(0, ROOT)
    import bench
    seen = set()
    for unit in ("sg_kernels.hip", "sg_colfs.hip"):
        _reached(unit, seen)
    assert {"bnd.hpp", "colw.hpp", "kcommon.hpp"} <= seen
    listed = {os.path.basename(f) for f in bench.KERNEL_SOURCES}
    assert seen <= listed, sorted(seen - listed)
    assert all(os.path.exists(os.path.join(ROOT, f)) for f in bench.KERNEL_SOURCES)
