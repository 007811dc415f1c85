"""GPU parity of the persistent batch kernel: batches of more than TDES_BATCH_TEAM_TILES tiles, which waves draw
from a work counter, under launch shapes and cut-overs of their own; and its build for the server's steps.

Every byte of the buffer is compared with plain launches of the same messages (other kernels), and blocks of
every message with the oracle.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs
from tests import _gpu
from tests.test_gpu_batch import _check_jobs, _layout, _table
from tests.test_gpu_serve import N_KEYS, _check_oracle, _outputs_by_tag, table  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu

# Two whole tiles and a remainder of 0 to 2047 blocks each: 2200 wave tiles or more under every cut-over.
LENGTHS = [4096 + 37 * j % 2048 for j in range(1100)]


@pytest.mark.parametrize("shape", [(64, 1, 0, 1), (64, 1, 0, 3), (128, 2, 1, 3), (256, 1, 2048, 2), (256, 6, 512, 16),
                                   (192, 3, 1800, 1)])
def test_shapes_and_replays_of_many_tiles(shape):
    """threads, workgroups per CU, cut-over, tiles per draw.  Every launch but the first relies on the counter
    that the one before it left at zero; one 64-thread workgroup per CU draws most tiles from it."""
    keys, table = _table(5, 0xC01)
    jobs, buf, total = _layout(LENGTHS, 0xC02)
    jobs["sched_idx"] = np.arange(jobs.size) % 5
    jobs["direction"] = np.arange(jobs.size) // 3 % 2
    ctx = td.tdes_ctx_create()
    try:
        td.tdes_ecb_batch(ctx, jobs, table, 5, buf, td.TDES_BATCH_PER_MESSAGE)
        torch.cuda.synchronize()
        want = buf.clone()
        _check_jobs(jobs, keys, want, 0xC02, sample_per_job=4)
        td.tdes_ctx_set_tuning(ctx, *shape)
        calls = [lambda: td.tdes_ecb_batch(ctx, jobs, table, 5, buf, td.TDES_BATCH_NO_GRAPH),
                 lambda: td.tdes_ecb_batch(ctx, jobs, table, 5, buf), lambda: td.tdes_ecb_batch_replay(ctx),
                 lambda: td.tdes_ecb_batch_replay(ctx), lambda: td.tdes_ecb_batch_replay(ctx, td.TDES_BATCH_NO_GRAPH)]
        for i, call in enumerate(calls):
            print(f"[persistent] shape {shape}, launch {i}", flush=True)
            buf[total: 2 * total].zero_()
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            assert torch.equal(buf, want), f"launch {i}"
            assert td.tdes_ctx_get_info(ctx)["tiles"] > td.TDES_BATCH_TEAM_TILES
    finally:
        td.tdes_ctx_destroy(ctx)


def test_tuned_server_steps_of_many_tiles(table):  # noqa: F811
    """Requests longer than TDES_BATCH_TEAM_TILES tiles, with short ones beside them, under a launch shape of
    the server's own: every block of every request against the oracle."""
    keys, dev_table = table
    reqs = np.zeros(12, dtype=td.REQUEST_DTYPE)
    reqs["n_blocks"] = [2048 * td.TDES_BATCH_TEAM_TILES + 1801, 700, 64, 5000, 2049, 1] * 2
    reqs["key_id"] = np.arange(12) * 41 % N_KEYS
    reqs["direction"] = [0] * 6 + [1] * 6
    reqs["seed"] = 0xC110 + np.arange(12)
    reqs["user_tag"] = np.arange(12)
    server = td.tdes_server_create(dev_table, N_KEYS, 1 << 30, max_inflight=2, max_step_jobs=8, max_step_blocks=1 << 24,
                                   keep_outputs=True, tuning=(128, 8, 1024, 2))
    try:
        print("[persistent] server steps of more than 2048 tiles", flush=True)
        done = td.tdes_server_run_trace(server, reqs, np.zeros(reqs.size))
        outs = _outputs_by_tag(server, done, reqs)
    finally:
        td.tdes_server_destroy(server)
    for i in range(reqs.size):
        _check_oracle(keys, reqs[i], outs[i])
