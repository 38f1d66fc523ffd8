"""The hash that ties a stored counter record to the kernels it was measured on
(CPU): every file of this package that a hashed source includes is hashed too, a
change of code changes it, one of comments or blank lines does not."""
import os
import re
import shutil
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402

CSRC = os.path.join(bench.ROOT, "paper_2003_03130_amd", "csrc")


def test_included_files_are_hashed():
    for fn in bench.TILE_KERNEL_SOURCES:
        with open(os.path.join(CSRC, fn)) as f:
            for inc in re.findall(r'#include "([^"]+)"', f.read()):
                # (the handle is host code)
                if os.path.exists(os.path.join(CSRC, inc)) and inc != "handle.h":
                    assert inc in bench.TILE_KERNEL_SOURCES, (fn, inc)


@pytest.mark.parametrize("fn", ["plate.h", "aux_kernels.h", "wide.hip", "prep.cpp"])
def test_code_counts_and_comments_do_not(tmp_path, fn):
    copy = str(tmp_path / "csrc")
    shutil.copytree(CSRC, copy)
    start = bench.kernel_source_hash(CSRC)
    assert bench.kernel_source_hash(copy) == start
    path = os.path.join(copy, fn)
    with open(path) as f:
        text = f.read()
    for extra, same in (("// a comment\n\n/* and\n another */\n", True),
                        ("static const char* s = \"// no comment\";\n", False),
                        ("int x;\n", False)):
        with open(path, "w") as f:
            f.write(extra + text)
        assert (bench.kernel_source_hash(copy) == start) is same
    with open(path, "w") as f:
        f.write(re.sub(r"//", "// more", text))
    assert bench.kernel_source_hash(copy) == start
