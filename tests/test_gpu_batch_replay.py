"""GPU parity of graphs that were captured behind one batch and replayed for another: of the same kind and within
the plan's buffer (the same graph, which takes its tile count from the plan), past it (a new graph, since the
buffer moved), and back to the first batch.

Every byte of the buffer is compared with plain launches of the replayed messages, and blocks of every message
with the oracle.  Tolerance: 0 bits.
"""
import numpy as np
import pytest
import torch

import paper_1305_4376_amd as td
from tests.test_gpu_batch import _check_jobs, _layout, _table

pytestmark = pytest.mark.gpu

# Per kind: the messages of a first batch, of one with more tiles in at most 8192 slots (the smallest plan
# buffer), and of one with more slots; 1799 blocks are 57 lane slots.
TILES = 2048
KINDS = {
    "a workgroup per tile": ([5000, 77, 2048], [TILES * 7] * 40 + [1799] * 30, [1799] * 400),
    "a wave per tile": ([TILES * 7] * 300 + [40], [TILES * 9] * 300 + [1799] * 20, [TILES * 8] * 300 + [1799] * 200),
}


@pytest.mark.parametrize("kind", KINDS)
def test_graphs_of_one_batch_replay_another(kind):
    batches = KINDS[kind]
    keys, table = _table(11, 0xC21)
    jobs, buf, total = _layout([n for lengths in batches for n in lengths], 0xC22)
    jobs["sched_idx"] = np.arange(jobs.size) % 11
    jobs["direction"] = np.arange(jobs.size) % 2
    ends = np.cumsum([len(lengths) for lengths in batches])
    parts = [jobs[end - len(lengths): end].copy() for end, lengths in zip(ends, batches)]
    ctx = td.tdes_ctx_create()
    try:
        for part, captures in ((0, 1), (1, 1), (2, 2), (0, 2)):
            print(f"[replay] {kind}: batch {part}", flush=True)
            buf[total: 2 * total].zero_()
            td.tdes_ecb_batch(ctx, parts[part], table, 11, buf, td.TDES_BATCH_PER_MESSAGE)
            torch.cuda.synchronize()
            want = buf.clone()
            _check_jobs(parts[part], keys, want, 0xC22, sample_per_job=4)
            td.tdes_ecb_batch(ctx, parts[part], table, 11, buf)
            info = td.tdes_ctx_get_info(ctx)
            assert (info["tiles"] <= td.TDES_BATCH_TEAM_TILES) == (kind == "a workgroup per tile")
            assert (info["slots"] > 8192) == (part == 2)
            for rep in range(3):
                buf[total: 2 * total].zero_()
                torch.cuda.synchronize()
                td.tdes_ecb_batch_replay(ctx)
                torch.cuda.synchronize()
                assert torch.equal(buf, want), f"batch {part}, replay {rep}"
            assert td.tdes_ctx_get_info(ctx)["graph_captures"] == captures, f"batch {part}"
    finally:
        td.tdes_ctx_destroy(ctx)
