"""GPU parity of the short-message kernel (one bit of f per lane, two blocks per wave).

Sizes at its edges: one block (half a wave), odd counts, a workgroup's eight blocks and one either
side, and the last size below each switch to another kernel with the one after it; ECB in both
directions, CTR with a counter that wraps inside the message, CBC decryption; 16- and 8-byte
aligned buffers; in place where the mode allows it.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu

pytestmark = pytest.mark.gpu

IV = b"\xff" * 7 + b"\xfd"  # the counter wraps after three blocks


@pytest.mark.parametrize("n", [1, 2, 3, 7, 8, 9, 255, 4097, 12287, 12288])
@pytest.mark.parametrize("offset", [0, 8])
def test_short_messages_match_oracle(n, offset):
    print(f"[short] n={n} offset={offset}", flush=True)
    keys = inputs.key_triple(inputs.KEY_SEED_BASE + 700 + n % 13)
    host = inputs.message(inputs.DATA_SEED_BASE + 700 + n, n)
    sched, src = _gpu.device_sched(*keys), _gpu.to_device(host, offset)
    guard = torch.full((8 * n + 16 + offset,), 0xA5, dtype=torch.uint8, device=_gpu.DEV)
    dst = guard[offset: offset + 8 * n]

    def check(want):
        torch.cuda.synchronize()
        assert np.array_equal(dst.cpu().numpy(), want)
        assert bool((guard[offset + 8 * n:] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())

    td.tdes_ecb_encrypt(sched, src, dst)
    check(oracle.tdes_ecb(*keys, host, decrypt=False, threads=_gpu.ORACLE_THREADS))
    td.tdes_ecb_decrypt(sched, src, dst)
    check(oracle.tdes_ecb(*keys, host, decrypt=True, threads=_gpu.ORACLE_THREADS))
    td.tdes_ctr_crypt(sched, IV, src, dst)
    check(oracle.tdes_ctr(*keys, IV, host))
    td.tdes_cbc_decrypt(sched, IV, src, dst)
    check(oracle.tdes_cbc(*keys, IV, host, decrypt=True))
    td.tdes_ecb_encrypt(sched, src, src)  # in place
    td.tdes_ecb_decrypt(sched, src, src)
    torch.cuda.synchronize()
    assert np.array_equal(src.cpu().numpy(), host)
