"""Every kernel that the sources define is in the built library (no GPU needed): the names come from the sources,
so that a kernel added later is looked for too, and are looked for as kernel descriptors, which only the embedded
gfx950 code has.
"""
import glob
import os
import re

import pytest

import paper_1305_4376_amd as td
from paper_1305_4376_amd import build

KERNEL = re.compile(r"__global__[^;{]*?\bvoid\s+(\w+)")


def _kernels():
    names = set()
    for path in glob.glob(os.path.join(build.CSRC, "*.hip")):
        text = re.sub(r"//.*|\\\n", "", open(path).read())
        found = KERNEL.findall(text)
        assert len(found) == text.count("__global__"), path
        names.update(found)
    return sorted(names)


@pytest.mark.parametrize("name", _kernels())
def test_the_library_has_the_kernel(name):
    data = open(td.library_path(), "rb").read()
    assert re.search(rf"_Z\w*{len(name)}{name}\w*\.kd\0".encode(), data), name  # mangled: the name behind its length


def test_every_source_is_built():
    assert _kernels()
    assert set(os.path.basename(p) for p in glob.glob(os.path.join(build.CSRC, "*.hip"))) <= set(build.SOURCES)
