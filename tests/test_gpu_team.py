"""GPU parity of the kernel that shares a tile of 2048 blocks between a workgroup's eight waves, and of
the switch from it to one wave per tile with a short partial tile behind the whole ones.

Sizes on both sides of its range in each mode, with a whole last tile, one of a single block and one
that lacks one block or ends inside a row of 64; 16- and 8-byte aligned buffers; a CTR counter that
wraps inside the message; in place where the mode allows it; bytes around the output untouched.
Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu

pytestmark = pytest.mark.gpu


def _case(seed, n, offset):
    keys = inputs.key_triple(inputs.KEY_SEED_BASE + seed)
    host = inputs.message(inputs.DATA_SEED_BASE + seed, n)
    guard = torch.full((8 * n + 16 + offset,), 0xA5, dtype=torch.uint8, device=_gpu.DEV)
    return keys, host, _gpu.device_sched(*keys), _gpu.to_device(host, offset), guard, guard[offset: offset + 8 * n]


def _check(guard, dst, offset, want):
    torch.cuda.synchronize()
    assert np.array_equal(dst.cpu().numpy(), want)
    assert bool((guard[offset + dst.numel():] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())


@pytest.mark.parametrize("n", [393215, 393216, 393217, 327679, 327680, 327681, 331000, 2097151, 2097152, 2097153, 2099199, 2359295, 2359296, 2359297, 2361343])
@pytest.mark.parametrize("offset", [0, 8])
def test_ecb_around_the_team_range(n, offset):
    print(f"[team] ecb n={n} offset={offset}", flush=True)
    keys, host, sched, src, guard, dst = _case(800 + n % 11, n, offset)
    idx = _gpu.sample_indices(n, 20000, 3, boundaries=range(0, n, 2048))
    want = {d: oracle.tdes_ecb(*keys, host.reshape(-1, 8)[idx].reshape(-1), decrypt=d, threads=_gpu.ORACLE_THREADS)
            for d in (False, True)}
    for decrypt, call in ((False, td.tdes_ecb_encrypt), (True, td.tdes_ecb_decrypt)):
        call(sched, src, dst)
        torch.cuda.synchronize()
        assert np.array_equal(_gpu.gather_blocks(dst, idx), want[decrypt])
        assert bool((guard[offset + 8 * n:] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())
    td.tdes_ecb_decrypt(sched, src, src)  # in place
    td.tdes_ecb_encrypt(sched, src, src)
    torch.cuda.synchronize()
    assert np.array_equal(src.cpu().numpy(), host)


@pytest.mark.parametrize("n", [393215, 393216, 393217, 395263, 45055, 45056, 45057, 47103, 47105, 49100])
@pytest.mark.parametrize("offset", [0, 8])
def test_modes_around_the_team_range(n, offset):
    print(f"[team] modes n={n} offset={offset}", flush=True)
    keys, host, sched, src, guard, dst = _case(820 + n % 11, n, offset)
    iv = (2**64 - n // 2).to_bytes(8, "big")  # the counter wraps in the middle
    td.tdes_ctr_crypt(sched, iv, src, dst)
    _check(guard, dst, offset, oracle.tdes_ctr(*keys, iv, host))
    td.tdes_cbc_decrypt(sched, iv, src, dst)
    _check(guard, dst, offset, oracle.tdes_cbc(*keys, iv, host, decrypt=True))
    td.tdes_ctr_crypt(sched, iv, src, src)  # in place
    td.tdes_ctr_crypt(sched, iv, src, src)
    torch.cuda.synchronize()
    assert np.array_equal(src.cpu().numpy(), host)


@pytest.mark.parametrize("n", [2359295, 2359296, 2359297, 2361343])
@pytest.mark.parametrize("offset", [0, 8])
def test_modes_of_long_messages(n, offset):
    """The first tiles and everything from two tiles before the end: a partial last tile is its own launch."""
    print(f"[team] long modes n={n} offset={offset}", flush=True)
    keys, host, sched, src, guard, dst = _case(840 + n % 11, n, offset)
    at = n // 2048 * 2048 - 4096
    iv = (2**64 - at - 5000).to_bytes(8, "big")  # the counter wraps near the end
    td.tdes_ctr_crypt(sched, iv, src, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    assert np.array_equal(got[: 8 * 4096], oracle.tdes_ctr(*keys, iv, host[: 8 * 4096]))
    iv_at = ((int.from_bytes(iv, "big") + at) % 2**64).to_bytes(8, "big")
    assert np.array_equal(got[8 * at:], oracle.tdes_ctr(*keys, iv_at, host[8 * at:]))
    td.tdes_cbc_decrypt(sched, iv, src, dst)
    torch.cuda.synchronize()
    got = dst.cpu().numpy()
    assert np.array_equal(got[: 8 * 4096], oracle.tdes_cbc(*keys, iv, host[: 8 * 4096], decrypt=True))
    assert np.array_equal(got[8 * at:], oracle.tdes_cbc(*keys, host[8 * at - 8: 8 * at].tobytes(), host[8 * at:], decrypt=True))
    assert bool((guard[offset + 8 * n:] == 0xA5).all()) and bool((guard[:offset] == 0xA5).all())
