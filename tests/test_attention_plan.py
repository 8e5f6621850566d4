"""How tree attention is cut into workgroups, on the host alone."""
import os

import pytest


def _plan(*a, **k):
    from paper_2401_12522_amd import binding, build
    if not os.path.exists(build.LIB_PATH):
        build.build_library()
    return binding.attention_plan_info(*a, **k)


@pytest.mark.parametrize("batch,rows,heads,kv_heads,ctx,expect", [
    (1, 68, 32, 32, 1024, dict(heads=1, rows=16, waves=8, workgroups=160, splits=1)),
    (4, 68, 32, 32, 1400, dict(heads=1, rows=16, waves=4, workgroups=640)),
    (1, 68, 64, 8, 2048, dict(heads=8, rows=4, waves=8, workgroups=136)),
    (8, 68, 64, 8, 4096, dict(heads=8, rows=4, waves=4, workgroups=1088)),
    (2, 40, 12, 2, 100, dict(heads=2, rows=16, waves=8)),           # six heads of a K/V head: pairs
    (2, 40, 24, 2, 100, dict(heads=4, rows=8)),
    (2, 40, 64, 2, 100, dict(heads=16, rows=2)),
    (1, 1, 32, 32, 4096, dict(heads=1, splits=8, workgroups=256, waves=8)),
])
def test_heads_rows_and_waves_of_a_workgroup(batch, rows, heads, kv_heads, ctx, expect):
    plan = _plan(batch, rows, heads, kv_heads, 128, ctx, n_prompt=16)
    assert {k: plan[k] for k in expect} == expect, plan


@pytest.mark.parametrize("batch,rows,heads,kv_heads,ctx,heads_wg", [
    # the pairs' workgroups fit an XCD's 32 CUs: up to 4 queries share a tile
    (1, 1, 64, 8, 2048, 8), (1, 2, 64, 8, 2048, 4), (1, 3, 64, 8, 2048, 2), (1, 5, 64, 8, 2048, 2), (4, 15, 64, 8, 2048, 2),
    (1, 2, 32, 8, 1000, 4), (1, 8, 32, 8, 1000, 2), (1, 1, 32, 1, 100, 8), (1, 3, 32, 1, 1000, 2),
    # they queue: as many as there are
    (1, 5, 32, 1, 4096, 16), (12, 5, 64, 8, 2048, 8), (70, 3, 24, 2, 33, 4),
    # but not where that leaves as many workgroups as before, as long as the rows are fewer than two tiles'
    (1, 9, 12, 1, 8000, 2), (1, 16, 64, 8, 2048, 2), (1, 17, 64, 8, 2048, 8), (2, 25, 12, 1, 2048, 2), (1, 32, 64, 8, 2048, 8),
])
def test_heads_share_a_tile_where_that_saves_time(batch, rows, heads, kv_heads, ctx, heads_wg):
    plan = _plan(batch, rows, heads, kv_heads, 128, ctx)
    assert plan["heads"] == heads_wg, plan
    assert plan["rows"] == 32 // heads_wg


@pytest.mark.parametrize("batch,rows,heads,kv_heads,ctx,page,waves", [
    (1, 136, 32, 32, 1024, 0, 4), (1, 128, 32, 32, 1024, 0, 8),                                    # more workgroups than CUs
    # two workgroups of four waves and their page tables in a CU's LDS: 3840 entries with two tiles, 3968 with one
    (1, 96, 64, 8, 61440, 16, 4), (1, 96, 64, 8, 61441, 16, 8), (1, 17, 32, 32, 63488, 16, 4), (1, 17, 32, 32, 63489, 16, 8),
    # an odd round of 256 at the end of long paged walks
    (4, 68, 32, 32, 1292, 64, 4), (4, 68, 32, 32, 1400, 64, 4), (4, 68, 32, 32, 1500, 64, 8), (4, 68, 32, 32, 1500, 0, 4), (2, 133, 32, 32, 5630, 16, 8),
    (2, 120, 32, 32, 5630, 16, 4), (3, 204, 32, 32, 1026, 16, 4), (5, 127, 32, 32, 4594, 16, 8), (8, 68, 64, 8, 2000, 64, 4),
    (1, 360, 64, 8, 5000, 64, 8),
    # and of long contiguous ones with one head per workgroup
    (1, 357, 32, 32, 5360, 0, 8), (1, 285, 32, 32, 6309, 0, 4), (1, 357, 32, 32, 2000, 0, 4), (1, 351, 64, 8, 6806, 0, 4), (1, 512, 32, 32, 5360, 0, 4),
])
def test_four_waves_where_two_workgroups_share_a_cu(batch, rows, heads, kv_heads, ctx, page, waves):
    plan = _plan(batch, rows, heads, kv_heads, 128, ctx, n_prompt=16, page_size=page)
    assert plan["waves"] == waves, plan


def _launch(*a, **k):
    from paper_2401_12522_amd import binding
    _plan(*a, **k)                                  # (builds the library where it is missing)
    return binding.attention_launch_info(*a, **k)


@pytest.mark.parametrize("batch,rows,heads,kv_heads,hd,ctx,page,share,waves,workgroups", [
    # two tiles where that saves a round or most of one, four where two would still queue
    (4, 68, 32, 32, 128, 900, 0, 2, 4, 384), (4, 68, 32, 32, 128, 1400, 64, 2, 4, 384), (5, 68, 32, 32, 128, 2200, 0, 2, 4, 480),
    (3, 100, 32, 32, 128, 900, 0, 2, 4, 384), (2, 256, 32, 32, 128, 1000, 0, 2, 4, 512), (8, 25, 40, 40, 128, 1000, 0, 2, 4, 320),
    (8, 68, 32, 32, 128, 900, 0, 4, 4, 512), (8, 68, 32, 32, 128, 100, 16, 4, 4, 512),
    (6, 68, 32, 32, 128, 900, 0, 1, 4, 960), (5, 100, 32, 32, 128, 2200, 0, 1, 4, 1120),
    # up to 640 single tiles only on walks of up to 51 chunks
    (4, 68, 32, 32, 128, 1456, 0, 2, 4, 384), (4, 68, 32, 32, 128, 1457, 0, 1, 4, 640), (3, 96, 32, 32, 128, 3000, 0, 1, 4, 576),
    (3, 68, 40, 40, 128, 2200, 0, 1, 4, 600), (4, 68, 40, 40, 128, 4096, 0, 2, 4, 480),
    # up to 512 single tiles do not queue, eight waves, pairs of heads, 64-wide heads and key splits never share
    (3, 68, 32, 32, 128, 900, 0, 1, 4, 480), (4, 68, 32, 32, 128, 1500, 64, 1, 8, 640), (8, 68, 64, 8, 128, 2000, 0, 1, 4, 1088),
    (32, 68, 4, 4, 64, 1000, 0, 1, 4, 640), (1, 1, 32, 32, 128, 4096, 0, 1, 8, 256),
    # one sequence: eight waves over four tiles where that leaves one round
    (1, 512, 32, 32, 128, 512, 0, 4, 8, 256), (1, 465, 32, 32, 128, 0, 64, 4, 8, 256), (1, 464, 32, 32, 128, 512, 0, 1, 4, 928),
    (1, 384, 40, 40, 128, 512, 0, 4, 8, 240), (1, 368, 40, 40, 128, 512, 0, 1, 4, 920), (1, 385, 40, 40, 128, 512, 0, 1, 4, 1000)])
def test_which_row_tiles_share_chunks(batch, rows, heads, kv_heads, hd, ctx, page, share, waves, workgroups):
    args, kw = (batch, rows, heads, kv_heads, hd, ctx), dict(n_prompt=16 if batch > 1 else 0, page_size=page)
    plan, launch = _plan(*args, **kw), _launch(*args, **kw)
    assert (launch["share"], launch["waves"], launch["workgroups"]) == (share, waves, workgroups), launch
    assert (launch["splits"], launch["heads"], launch["rows"]) == (plan["splits"], plan["heads"], share * plan["rows"])
    if share == 1:
        assert all(launch[k] == plan[k] for k in plan)


@pytest.mark.parametrize("batch,rows,heads,kv_heads,hd,ctx,page,ranked", [
    (8, 68, 64, 8, 128, 4096, 0, True), (8, 68, 64, 8, 64, 4096, 64, True), (2, 170, 64, 8, 128, 3000, 0, True), (8, 130, 16, 2, 64, 3000, 0, True),
    (8, 68, 64, 8, 128, 1841, 0, True), (8, 68, 64, 8, 128, 1840, 0, False),                     # 64 chunks
    (9, 68, 64, 8, 128, 4096, 0, False), (3, 68, 64, 8, 128, 4096, 0, False), (1, 300, 64, 8, 128, 4096, 0, False),   # one lane a pair; no queue
    (8, 68, 64, 1, 128, 4096, 0, False), (4, 137, 32, 2, 128, 4096, 0, False),                   # an XCD walks one sequence only
    (8, 68, 64, 8, 128, 20000, 0, False), (4, 68, 32, 32, 128, 4096, 0, False)])                 # key splits, single heads
def test_sequences_start_longest_first_on_long_walks_that_queue(batch, rows, heads, kv_heads, hd, ctx, page, ranked):
    launch = _launch(batch, rows, heads, kv_heads, hd, ctx, n_prompt=16, page_size=page)
    assert launch["ranked"] is ranked, launch


def test_plans_of_nothing_are_refused():
    from paper_2401_12522_amd import binding
    for bad in ((0, 1, 4, 4, 64, 0), (1, 1, 4, 3, 64, 0), (1, 1, 4, 4, 96, 0), (1, 1, 4, 4, 64, -1)):
        with pytest.raises(binding.BitaError, match="bita_attention_plan_info"):
            _plan(*bad)
        with pytest.raises(binding.BitaError, match="bita_attention_launch_info"):
            binding.attention_launch_info(*bad)
