"""The loads of a tile are in flight together, also where each of them hangs on a condition (partial wave tiles and
lane tiles, eight at a time): read from the assembly that the kernels are compiled to (no GPU needed).  A wave that waits for each of
its 32 loads before it issues the next has 32 trips to memory one after the other.
"""
import os
import re
import subprocess

import pytest

from paper_1305_4376_amd import build


def _waited_at_once(text, kernel):
    """Loads of a kernel, and how many of them are waited for before the next one."""
    body = re.search(rf"^_ZN12_GLOBAL__N_1{len(kernel)}{kernel}E\w*:.*?^\.Lfunc_end", text, re.S | re.M).group(0)
    loads = waited = 0
    pending = False
    for line in body.splitlines():
        op = line.strip()
        if op.startswith("global_load"):
            loads, pending = loads + 1, True
        elif op.startswith("s_waitcnt") and "vmcnt(0)" in op:
            waited += pending
            pending = False
    return loads, waited


@pytest.mark.parametrize("source, kernel, tile_loads", [("k_batch.hip", "tdes_batch_kernel", 80),
                                                        ("k_static.hip", "tdes_static_batch_kernel", 48),
                                                        ("k_bitslice.hip", "tdes_bitslice_tail_kernel", 32)])
def test_tile_loads_do_not_wait_for_each_other(source, kernel, tile_loads, tmp_path):
    out = tmp_path / "kernel.s"
    subprocess.check_call([build.HIPCC, *build.COMMON, "-x", "hip", "--cuda-device-only", "-S", "-o", str(out),
                           os.path.join(build.CSRC, source)], stderr=subprocess.DEVNULL)
    loads, waited = _waited_at_once(out.read_text(), kernel)
    assert loads >= tile_loads
    assert 4 * waited <= loads, f"{waited} of {loads}"  # counters, slots, key words, and the last of every group of loads
