"""GPU parity of the table kernel with two lanes per block, and of the switches to and from it.

Sizes at both ends of its ranges and inside them: odd counts, a workgroup's 128 and 256 blocks and one either
side, the last size that one pass of the resident workgroups covers and the next; ECB in both directions, CTR
with a counter that wraps inside the message, CBC decryption; 16- and 8-byte aligned buffers; in place where
the mode allows it; bytes around the output untouched.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu

pytestmark = pytest.mark.gpu

SIZES = [12287, 12288, 12289, 12417, 90112, 90113, 131072, 131073, 262144, 262145, 262401, 393216, 393217]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("offset", [0, 8])
def test_pair_messages_match_oracle(n, offset):
    print(f"[pair] n={n} offset={offset}", flush=True)
    keys = inputs.key_triple(inputs.KEY_SEED_BASE + 950 + n % 13)
    host = inputs.message(inputs.DATA_SEED_BASE + 950 + n, n)
    sched, src = _gpu.device_sched(*keys), _gpu.to_device(host, offset)
    guard = torch.full((8 * n + 16 + offset,), 0xA5, dtype=torch.uint8, device=_gpu.DEV)
    dst = guard[offset: offset + 8 * n]

    def check(want, first=0):
        torch.cuda.synchronize()
        assert np.array_equal(dst.cpu().numpy()[8 * first: 8 * first + want.size], want)
        assert bool((guard[offset + 8 * n:] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())

    td.tdes_ecb_encrypt(sched, src, dst)
    check(oracle.tdes_ecb(*keys, host, decrypt=False, threads=_gpu.ORACLE_THREADS))
    td.tdes_ecb_decrypt(sched, src, dst)
    check(oracle.tdes_ecb(*keys, host, decrypt=True, threads=_gpu.ORACLE_THREADS))
    iv = (2**64 - n + 1000).to_bytes(8, "big")  # the counter wraps 1000 blocks before the end
    for first in (0, n // 2, n - 4096):  # the modes' oracle runs on one thread: three windows of the message
        part, at = host[8 * first: 8 * (first + 4096)], ((int.from_bytes(iv, "big") + first) % 2**64).to_bytes(8, "big")
        td.tdes_ctr_crypt(sched, iv, src, dst)
        check(oracle.tdes_ctr(*keys, at, part), first)
        td.tdes_cbc_decrypt(sched, iv, src, dst)
        before = host[8 * first - 8: 8 * first].tobytes() if first else iv
        check(oracle.tdes_cbc(*keys, before, part, decrypt=True), first)
    td.tdes_ecb_encrypt(sched, src, src)  # in place
    td.tdes_ctr_crypt(sched, iv, src, src)
    td.tdes_ctr_crypt(sched, iv, src, src)
    td.tdes_ecb_decrypt(sched, src, src)
    torch.cuda.synchronize()
    assert np.array_equal(src.cpu().numpy(), host)
