"""Workloads of the library as its users run them, for timing one build against another.

Every case is one call through the Python binding's public entry points on data that is already
in GPU memory: messages of uniform random bytes (what ciphertext is, and what the cost does not
depend on), key triples with odd parity, schedules expanded and uploaded beforehand.  `listed()`
names the cases, `draw(rng)` gives others of the same ranges, `prepare` makes what the program
holds before the call, `run` is the call, `work` is what it cannot do without.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1305_4376_amd as td
from paper_1305_4376_amd import inputs

# 32-bit logic operations per block that the bitsliced algorithm needs: per round 48 key XORs, a
# 209-gate S-box layer and 32 XORs into the other half, for 32 blocks at a time, over 48 rounds.
OPS_PER_BLOCK = 48 * (48 + 209 + 32) / 32


def listed():
    return [
        # One message, ECB.
        # A short record (a database field, a network packet train): the smallest call, all latency.
        {"name": "ecb_enc_2KiB", "call": "ecb", "blocks": 256, "decrypt": False, "keying": 3, "offset": 0},
        # A 64 KiB message under a two-key triple, the smallest message of the benchmark's size sweep.
        {"name": "ecb_dec_64KiB", "call": "ecb", "blocks": 8192, "decrypt": True, "keying": 2, "offset": 0},
        # The 1 MiB message: the paper's own chunk, and the benchmark's single-message latency figure.
        {"name": "ecb_enc_1MiB", "call": "ecb", "blocks": 131072, "decrypt": False, "keying": 3, "offset": 0},
        # 4 MiB, the size sweep's second message: a file or a block of a store.
        {"name": "ecb_dec_4MiB", "call": "ecb", "blocks": 524288, "decrypt": True, "keying": 3, "offset": 0},
        # A ragged 24 MB message behind an 8-byte header, as a file with a length word in front arrives.
        {"name": "ecb_enc_24MB_ragged", "call": "ecb", "blocks": 3000001, "decrypt": False, "keying": 3, "offset": 8},
        # The headline: one 1 GiB message resident in HBM.
        {"name": "ecb_enc_1GiB", "call": "ecb", "blocks": 1 << 27, "decrypt": False, "keying": 3, "offset": 0},
        # The block-parallel modes.
        # CTR over a short message that is not a whole tile: a request or a packet burst.
        {"name": "ctr_64KB_ragged", "call": "ctr", "blocks": 8001, "decrypt": False, "keying": 3, "offset": 0},
        # CTR over a 16 MB message.
        {"name": "ctr_16MB", "call": "ctr", "blocks": 2000000, "decrypt": False, "keying": 3, "offset": 0},
        # CBC decryption of a 256 MiB archive, the size sweep's third message.
        {"name": "cbc_dec_256MiB", "call": "cbc", "blocks": 1 << 25, "decrypt": True, "keying": 3, "offset": 0},
        # Many messages, each under its own key triple.
        # A light serving step: a few dozen requests of 512 B to 1 MiB, half of them decryptions.
        {"name": "batch_48_requests", "call": "batch", "messages": 48, "min_blocks": 64, "max_blocks": 131072},
        # The benchmark's batch: 4096 messages of 1 .. 131072 blocks, planned, uploaded and launched.
        {"name": "batch_4096_messages", "call": "batch", "messages": 4096, "min_blocks": 1, "max_blocks": 131072},
        # The allocation-free batch: 512 records of up to 64 KiB, the jobs already on the device.
        {"name": "static_512_records", "call": "static", "messages": 512, "min_blocks": 1, "max_blocks": 8192},
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of lo .. hi."""
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    call = rng.choice(["ecb", "ecb", "ecb", "ctr", "cbc", "batch", "static"])
    if call in ("ecb", "ctr", "cbc"):
        blocks = _log_int(rng, 1, 1 << 26)
        if rng.random() < 0.3:  # a power of two, as buffers often are
            blocks = 1 << (blocks.bit_length() - 1)
        return {"call": call, "blocks": blocks, "decrypt": call == "cbc" or (call == "ecb" and rng.random() < 0.5),
                "keying": rng.choice([3, 3, 2, 1]), "offset": rng.choice([0, 0, 0, 8])}
    messages = _log_int(rng, 1, 4096 if call == "batch" else 2048)
    top = rng.choice([1024, 8192, 131072]) if call == "batch" else rng.choice([256, 2048, 8192])
    return {"call": call, "messages": messages, "min_blocks": rng.choice([1, 64]), "max_blocks": top}


def _lengths(case):
    """The batch's message lengths, log-uniform; a function of the case alone, so that every seed does the same work."""
    lo, hi, n = case["min_blocks"], case["max_blocks"], case["messages"]
    u = (inputs.splitmix64(inputs.DATA_SEED_BASE + 4, 0, n) >> np.uint64(11)).astype(np.float64) / (1 << 53)
    return np.clip(np.floor(lo * np.exp(u * np.log((hi + 1.0) / lo))).astype(np.int64), lo, hi)


def _upload(host):
    dev = torch.empty(host.size, dtype=torch.uint8, device="cuda")
    td.tdes_sched_upload(host, dev)
    return dev


class _Batch:
    """What a batching program keeps: the context, the schedule table, the jobs and the buffer."""

    def __init__(self, case, seed):
        lengths = _lengths(case)
        n = case["messages"]
        keys = inputs.key_triples(seed + 1, n)
        table = np.concatenate([td.tdes_expand_key(k[:8].tobytes(), k[8:16].tobytes(), k[16:].tobytes()) for k in keys])
        self.n, self.table = n, _upload(table)
        self.total = int(lengths.sum()) * 8
        self.buf = torch.zeros(2 * self.total, dtype=torch.uint8, device="cuda")
        td.tdes_fill_splitmix64(self.buf, self.total // 8, seed)
        self.out = self.buf[self.total:]
        jobs = np.zeros(n, dtype=td.JOB_DTYPE)
        starts = np.concatenate([[0], np.cumsum(lengths)[:-1]]) * 8
        jobs["in_off"], jobs["out_off"], jobs["n_blocks"] = starts, starts + self.total, lengths
        jobs["sched_idx"] = np.arange(n)
        jobs["direction"] = inputs.splitmix64(seed + 2, 0, n) & np.uint64(1)
        self.jobs, self.ctx = jobs, None
        if case["call"] == "batch":
            self.ctx = td.tdes_ctx_create()
        else:
            self.dev_jobs = torch.from_numpy(jobs.view(np.uint8).copy()).cuda()
            self.rejected = torch.zeros(1, dtype=torch.int32, device="cuda")

    def __del__(self):
        if getattr(self, "ctx", None):
            td.tdes_ctx_destroy(self.ctx)


def prepare(case, seed):
    call = case["call"]
    if call in ("batch", "static"):
        return call, _Batch(case, seed)
    n, off = case["blocks"], case["offset"]
    sched = _upload(td.tdes_expand_key(*inputs.key_triple(seed + 1, case["keying"])))
    src = torch.empty(8 * n + off, dtype=torch.uint8, device="cuda")[off:]
    dst = torch.zeros(8 * n + off, dtype=torch.uint8, device="cuda")[off:]
    td.tdes_fill_splitmix64(src, n, seed)
    iv = inputs.message(seed + 3, 1).tobytes()
    return call, (sched, src, dst, iv, case["decrypt"])


def run(state):
    call, s = state
    if call == "batch":
        td.tdes_ecb_batch(s.ctx, s.jobs, s.table, s.n, s.buf)
        return s.out
    if call == "static":
        td.tdes_ecb_batch_static(s.dev_jobs, s.n, s.table, s.n, s.buf, dev_rejected=s.rejected)
        return s.out, s.rejected
    sched, src, dst, iv, decrypt = s
    if call == "ctr":
        td.tdes_ctr_crypt(sched, iv, src, dst)
    elif call == "cbc":
        td.tdes_cbc_decrypt(sched, iv, src, dst)
    elif decrypt:
        td.tdes_ecb_decrypt(sched, src, dst)
    else:
        td.tdes_ecb_encrypt(sched, src, dst)
    return dst


def work(case):
    if case["call"] in ("batch", "static"):
        n, keys = int(_lengths(case).sum()), case["messages"]
    else:
        n, keys = case["blocks"], 1
    # every block read once and written once, and one direction's half of each schedule
    return {"bytes": 16 * n + keys * td.TDES_SCHED_BYTES // 2, "flops": n * OPS_PER_BLOCK}
