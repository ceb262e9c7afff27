"""The sources whose hash guards recorded HBM traffic figures (CPU): the
substitution kernels' file and every header of csrc/ it takes in, directly or
through another, so that a change to any of them makes the figures stale."""

import os
import re

from paper_1801_08655_amd import rocprof_summary as rs


def test_every_included_header_is_hashed():
    csrc = os.path.join(rs.HERE, "csrc")
    todo, seen = ["kernels_solve.hip"], set()
    while todo:
        f = todo.pop()
        if f in seen or not os.path.exists(os.path.join(csrc, f)):
            continue
        seen.add(f)
        with open(os.path.join(csrc, f)) as fh:
            todo += re.findall(r'^#include "([^"/]+)"', fh.read(), re.M)   # (csrc/ only)
    assert "kernels_tile.h" in seen
    assert {"csrc/" + f for f in seen} == set(rs.KERNEL_SOURCES)
