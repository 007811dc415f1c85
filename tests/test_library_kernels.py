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


def _vgprs(name):
    """A kernel's vector registers, from the metadata of the embedded code (msgpack, keys in order), as a wave is
    given them: in eights."""
    data = open(td.library_path(), "rb").read()
    found = re.findall(rf"{len(name)}{name}E\w*\.kd.{{0,400}}?\.vgpr_count(?:([\0-\x7f])|\xcc(.))".encode("latin-1"), data, re.S)
    assert len(found) == 1, (name, len(found))
    return -(-ord(found[0][0] or found[0][1]) // 8) * 8


@pytest.mark.parametrize("name, waves", [("tdes_plan_kernel", 1), ("fill_tiles_kernel", 2)])
def test_the_servers_small_kernels_fit_beside_its_cipher(name, waves):
    """Four waves of the capped batch kernel stay on every SIMD (512 registers a lane) until their step is done; the
    fills and plans of the next steps run in what they leave."""
    assert 4 * _vgprs("tdes_batch_kernel_capped") + waves * _vgprs(name) <= 512
