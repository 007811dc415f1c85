"""GPU parity of batches on both sides of the switch between a workgroup per tile and a wave per tile,
and of the plan that the device writes.

Batches of 1600 and 2048 tiles and of one more, only lane tiles (with idle lanes in the last one), only whole tiles, one
message long enough for several planning workgroups, messages whose last partial tile is a wave tile, and
empty messages between others, and both sides of the allocation-free batch's single launch; through tdes_ecb_batch (launched and replayed from its graph) and
tdes_ecb_batch_static.  Expected output: the oracle's on every block of short messages and on the ends and
a sample of long ones.  Bytes between the messages stay untouched.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu

pytestmark = pytest.mark.gpu

N_KEYS = 7
SHAPES = {
    "1600 whole tiles": [2048 * 4] * 400,
    "1601 tiles": [2048 * 4] * 400 + [1900],
    "2048 whole tiles": [2048 * 4] * 512,
    "2049 tiles": [2048 * 4] * 512 + [1900],
    "one lane": [5],
    "lane tiles, the last with idle lanes": [1, 31, 32, 33, 64, 1799] * 40,
    "wave remainders": [1800, 2047, 2048, 2049, 4096 + 1801],
    "one long message": [2048 * 700 + 77],
    "empty messages": [0, 40, 0, 0, 2048, 0],
    "4096 jobs, one launch": [j % 40 for j in range(4096)],
    "4097 jobs": [j % 40 for j in range(4097)],
    "65537 jobs": [1] * 65537,  # one record more than the plan's largest grid reads at a time
    "1500 tiles, mixed": [2048 + 64 * (j % 30) for j in range(1000)],
}


def _layout(lengths, seed):
    """Inputs, then outputs, 8 guard bytes behind each message; odd block offsets; both directions."""
    lengths = np.asarray(lengths, dtype=np.int64)
    room = (lengths + 1) * 8
    starts = np.concatenate([[0], np.cumsum(room)[:-1]])
    total = int(room.sum())
    jobs = np.zeros(lengths.size, dtype=td.JOB_DTYPE)
    jobs["in_off"], jobs["out_off"], jobs["n_blocks"] = starts, starts + total, lengths
    jobs["sched_idx"] = np.arange(lengths.size) % N_KEYS
    jobs["direction"] = (np.arange(lengths.size) // 2) % 2
    buf = torch.full((2 * total,), 0xA5, dtype=torch.uint8, device=_gpu.DEV)
    td.tdes_fill_splitmix64(buf, total // 8, seed)
    return jobs, buf, total


def _check(jobs, keys, buf, total, seed):
    torch.cuda.synchronize()
    host = buf.cpu().numpy()
    src = inputs.message(seed, total // 8)
    want = np.full(total, 0xA5, dtype=np.uint8)
    seen = np.ones(total, dtype=bool)
    for j, job in enumerate(jobs):
        n, lo, k = int(job["n_blocks"]), int(job["in_off"]), keys[job["sched_idx"]]
        idx = np.arange(n)
        if n > 4096:
            idx = np.unique(np.concatenate([idx[:256], idx[-2300:], np.random.default_rng(j).integers(0, n, 256)]))
            seen[lo: lo + 8 * n] = False
        if n == 0:
            continue
        pos = (lo + 8 * idx[:, None] + np.arange(8)).reshape(-1)
        want[pos] = oracle.tdes_ecb(k[:8].tobytes(), k[8:16].tobytes(), k[16:].tobytes(), src[pos],
                                    decrypt=bool(job["direction"]), threads=1)
        seen[pos] = True
    assert np.array_equal(host[total:][seen], want[seen])


@pytest.mark.parametrize("shape", SHAPES)
def test_batches_by_tiles(shape):
    print(f"[tiles] {shape}", flush=True)
    keys = inputs.key_triples(inputs.KEY_SEED_BASE + 900, N_KEYS)
    host = np.concatenate([td.tdes_expand_key(k[:8].tobytes(), k[8:16].tobytes(), k[16:].tobytes()) for k in keys])
    table = torch.empty(host.size, dtype=torch.uint8, device=_gpu.DEV)
    td.tdes_sched_upload(host, table)
    seed = inputs.DATA_SEED_BASE + 900
    jobs, buf, total = _layout(SHAPES[shape], seed)
    ctx = td.tdes_ctx_create()
    try:
        td.tdes_ecb_batch(ctx, jobs, table, N_KEYS, buf)
        _check(jobs, keys, buf, total, seed)
        info = td.tdes_ctx_get_info(ctx)
        assert info["blocks"] == int(jobs["n_blocks"].sum()) and info["tiles"] == info["wave_tiles"] + info["lane_tiles"]
        buf[total:].fill_(0xA5)
        td.tdes_ecb_batch_replay(ctx)
        _check(jobs, keys, buf, total, seed)
    finally:
        td.tdes_ctx_destroy(ctx)
    if jobs.size > td.TDES_STATIC_MAX_JOBS:
        return
    buf[total:].fill_(0xA5)
    dev_jobs = torch.from_numpy(jobs.view(np.uint8).copy()).to(_gpu.DEV)
    rejected = torch.ones(1, dtype=torch.int32, device=_gpu.DEV)
    td.tdes_ecb_batch_static(dev_jobs, jobs.size, table, N_KEYS, buf, dev_rejected=rejected)
    _check(jobs, keys, buf, total, seed)
    assert int(rejected.item()) == 0
