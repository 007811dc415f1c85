"""The batch tuner times only axes that the batch's kernel has (no GPU): a batch of at most
TDES_BATCH_TEAM_TILES tiles has a workgroup per tile, whatever the launch shape and the tiles per draw.
"""
import os
import re

import pytest
import torch

import paper_1305_4376_amd as td
from paper_1305_4376_amd import autotune

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class _Library:
    """A context that plans `tiles[cut-over]` tiles and forgets the rest."""

    TDES_BATCH_TEAM_TILES = td.TDES_BATCH_TEAM_TILES

    def __init__(self, tiles):
        self.tiles, self.tuning, self.planned = tiles, (256, 4, 1800, 1), None

    def tdes_ctx_set_tuning(self, ctx, threads, groups_per_cu, wave_remainder=0, tiles_per_draw=0):
        self.tuning = threads, groups_per_cu, wave_remainder or 1800, tiles_per_draw or 1

    def tdes_ecb_batch(self, *args):
        self.planned = self.tiles.get(self.tuning[2], self.tiles[None])

    def tdes_ctx_get_info(self, ctx):
        return dict(zip(autotune.FIELDS, self.tuning), tiles=self.planned, blocks=1 << 20)


def _tune(monkeypatch, tiles):
    timed = []

    def time_replays(ctx, tuning, reps):
        timed.append(tuning)
        return float(len(timed))

    monkeypatch.setattr(autotune, "td", _Library(tiles))
    monkeypatch.setattr(autotune, "_time_replays", time_replays)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    return timed, autotune.tune_batch(1, None, None, 1, None, path=None)


def test_few_tiles_time_the_cut_over_alone(monkeypatch):
    timed, result = _tune(monkeypatch, {None: td.TDES_BATCH_TEAM_TILES})
    assert timed == [(256, 4, rem, autotune.TILES_PER_DRAW[0]) for rem in autotune.WAVE_REMAINDER]
    assert (result["threads"], result["groups_per_cu"], result["tiles_per_draw"]) == (256, 4, 1)


def test_many_tiles_time_every_axis(monkeypatch):
    timed, _ = _tune(monkeypatch, {None: td.TDES_BATCH_TEAM_TILES + 1})
    shapes = len(autotune.THREADS) * len(autotune.GROUPS_PER_CU)
    assert len(timed) == shapes + len(autotune.WAVE_REMAINDER) * len(autotune.TILES_PER_DRAW)
    assert len(set(timed)) == len(timed)


def test_a_cut_over_that_leaves_few_tiles_is_timed_once(monkeypatch):
    timed, _ = _tune(monkeypatch, {None: td.TDES_BATCH_TEAM_TILES + 1, 2048: td.TDES_BATCH_TEAM_TILES})
    assert [t[3] for t in timed if t[2] == 2048] == [autotune.TILES_PER_DRAW[0]]


@pytest.mark.parametrize("name", ["TDES_BATCH_TEAM_TILES", "TDES_STATIC_MAX_JOBS"])
def test_the_bindings_limits_are_the_headers(name):
    header = open(os.path.join(ROOT, "include", "tdes.h")).read()
    assert int(re.search(rf"#define {name} (\d+)", header).group(1)) == getattr(td, name)
