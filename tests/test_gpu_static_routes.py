"""GPU parity of the allocation-free batch on each of its routes, with jobs it must refuse first, in the middle
and last, and with a plan of an earlier, larger call left in its scratch array.

Routes: one launch (also with 512 jobs, from where on its threads take several, and with more than the 2048 that are
read at a time); one launch that finds few tiles in a large buffer; at most 4096 jobs with more tiles than teams take (the first launch leaves a plan for the second); more than 4096 jobs (a plan kernel).  Every byte of the
buffer is compared with plain launches of the accepted messages, and the count of the refused ones.  Tolerance:
0 bits.
"""
import numpy as np
import pytest
import torch

import paper_1305_4376_amd as td
from tests.test_gpu_batch import _check_jobs, _layout, _table

pytestmark = pytest.mark.gpu

N_KEYS = 9
SEED = 0xC32
ROUTES = {
    "one launch": ([3000, 100, 2048, 77, 5000, 64, 1] * 4, 0),
    "512 jobs, one for each thread": ([1 + j % 70 for j in range(512)], 0),
    "513 jobs": ([1 + j % 70 for j in range(513)], 0),
    "2049 jobs, more than are read at a time": ([1 + j % 40 for j in range(2049)], 0),
    "few tiles in a large buffer": ([3000, 100, 2048, 77, 5000, 64, 1] * 4, 48 << 20),
    "two launches, one plans": ([2049 + 5 * j for j in range(1000)], 0),
    "a plan kernel": ([1 + j % 90 for j in range(4200)], 0),
}


def _refuse(jobs, table_bytes):
    """A copy of the jobs with every kind of malformed one, in runs at both ends and in the middle."""
    bad = jobs.copy()
    n = jobs.size
    which = [0, 1, n // 2 - 2, n // 2 - 1, n // 2, n // 2 + 1, n - 2, n - 1]
    bad["sched_idx"][which[0]] = N_KEYS                        # no such schedule
    bad["direction"][which[1]] = 2                             # no such direction
    bad["in_off"][which[2]] = table_bytes                      # reads past the buffer
    bad["out_off"][which[3]] = table_bytes - 8                 # writes past it (two blocks at least)
    bad["n_blocks"][which[3]] = 2
    bad["in_off"][which[4]] += 4                               # misaligned
    bad["out_off"][which[5]] = bad["in_off"][which[5]] + 8     # overlaps itself
    bad["n_blocks"][which[5]] = 2
    bad["n_blocks"][which[6]] = (1 << 40) + 1                  # too long
    bad["out_off"][which[7]] = 2 ** 64 - 8                     # offset arithmetic would wrap
    return bad, np.setdiff1d(np.arange(n), which), len(which)


def _call(jobs, table, buf):
    dev_jobs = torch.from_numpy(jobs.view(np.uint8).copy()).to(buf.device)
    rejected = torch.full((1,), -1, dtype=torch.int32, device=buf.device)
    td.tdes_ecb_batch_static(dev_jobs, jobs.size, table, N_KEYS, buf, dev_rejected=rejected)
    torch.cuda.synchronize()
    return int(rejected.item())


def _plain(jobs, table, buf):
    ctx = td.tdes_ctx_create()
    try:
        td.tdes_ecb_batch(ctx, jobs, table, N_KEYS, buf, td.TDES_BATCH_PER_MESSAGE)
        torch.cuda.synchronize()
    finally:
        td.tdes_ctx_destroy(ctx)
    return buf


def _prepare(route):
    lengths, more = ROUTES[route]
    keys, table = _table(N_KEYS, 0xC31)
    jobs, buf, total = _layout(lengths, SEED, in_place_every=4)
    jobs["sched_idx"] = np.arange(jobs.size) % N_KEYS
    jobs["direction"] = np.arange(jobs.size) // 2 % 2
    buf[2 * total:].zero_()
    buf[total: 2 * total].zero_()
    return keys, table, jobs, torch.cat([buf, torch.zeros(more, dtype=torch.uint8, device=buf.device)])


@pytest.mark.parametrize("route", ROUTES)
def test_refused_jobs_by_route(route):
    print(f"[static] {route}: refused jobs", flush=True)
    keys, table, jobs, buf = _prepare(route)
    bad, good, refused = _refuse(jobs, buf.numel())
    want = _plain(jobs[good], table, buf.clone())
    assert _call(bad, table, buf) == refused
    assert torch.equal(buf, want)
    _check_jobs(jobs[good], keys, buf, SEED, sample_per_job=4)
    # every job refused
    bad["direction"] = 2
    assert _call(bad, table, buf) == jobs.size
    assert torch.equal(buf, want)


@pytest.mark.parametrize("second", ["two launches, one plans", "a plan kernel"])
@pytest.mark.parametrize("first", ["two launches, one plans", "a plan kernel"])
def test_an_earlier_plan_is_not_seen(first, second):
    """A larger call by `first`, then one by `second` with the same jobs' odd ones and a tail left out: nothing
    else may be written by it."""
    print(f"[static] {second} after {first}", flush=True)
    _, table, jobs, buf = _prepare(first)
    want = _plain(jobs, table, buf.clone())
    assert _call(jobs, table, buf) == 0
    assert torch.equal(buf, want)
    _, table, jobs, buf = _prepare(second)
    if second == "a plan kernel":
        jobs = jobs[:4100]                # still more than 4096
        jobs["n_blocks"][::2] = 0
    else:
        jobs = jobs[:900]                 # still more than 1600 tiles
        jobs["n_blocks"][::50] = 0
    want = _plain(jobs, table, buf.clone())
    assert _call(jobs, table, buf) == 0
    assert torch.equal(buf, want)
