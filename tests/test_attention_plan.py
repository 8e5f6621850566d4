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


def test_plans_of_nothing_are_refused():
    from paper_2401_12522_amd import binding
    for bad in ((0, 1, 4, 4, 64, 0), (1, 1, 4, 3, 64, 0), (1, 1, 4, 4, 96, 0), (1, 1, 4, 4, 64, -1)):
        with pytest.raises(binding.BitaError, match="bita_attention_plan_info"):
            _plan(*bad)
