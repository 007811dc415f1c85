"""GPU parity of the table kernel on both sides of every length at which its workgroup size changes (256 threads to
2^16 blocks, in most of the first half of its second and fourth pass, else 512), asked for by name; both alignments.
Expected output: the oracle's on every block.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu

pytestmark = pytest.mark.gpu

EDGES = [1 << 16, 1 << 18, (1 << 18) + 1024, 3 << 17, (3 << 18) + 1024, 7 << 17]
N = max(EDGES) + 1


@pytest.fixture(scope="module")
def message():
    keys = inputs.key_triple(inputs.KEY_SEED_BASE + 930)
    host = inputs.message(inputs.DATA_SEED_BASE + 930, N)
    return _gpu.device_sched(*keys), host, oracle.tdes_ecb(*keys, host, threads=_gpu.ORACLE_THREADS)


@pytest.mark.parametrize("offset", [0, 8])
@pytest.mark.parametrize("edge", EDGES)
def test_table_kernel_at_its_switches(message, edge, offset):
    sched, host, want = message
    for n in (edge - 1, edge, edge + 1):
        print(f"[table] n={n} offset={offset}", flush=True)
        src = _gpu.to_device(host[: 8 * n], offset)
        guard = torch.full((8 * n + 16 + offset,), 0xA5, dtype=torch.uint8, device=_gpu.DEV)
        dst = guard[offset: offset + 8 * n]
        _gpu.run(sched, src, dst, n, td.TDES_ENCRYPT, td.TDES_VARIANT_TABLE)
        assert np.array_equal(dst.cpu().numpy(), want[: 8 * n])
        assert bool((guard[offset + 8 * n:] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())
        _gpu.run(sched, dst, dst, n, td.TDES_DECRYPT, td.TDES_VARIANT_TABLE)  # in place
        assert bool((dst == src).all())
