"""A batch emits each program's code again: with the options its plan was
made with, so that its tile's workspace and LDS, sized from the plan, hold
what the code stores."""

import re

import pytest

import paper_2408_09662_amd as xg
from tests import plan_probe
from workloads import configs
from workloads.ldl import ldl_solve


def accesses(src, es):
    """(largest workspace byte offset of a slot, the tile's workspace bytes)"""
    used = max((int(o) for o in re.findall(r"xg_w(?:ld|st)\(wsr, (\d+)u", src)), default=-1)
    have = [int(v) * es for v in re.findall(r"\(short\)0, \(int\)\((\d+) \* sizeof\(T\)\)", src)]
    assert len(set(have)) <= 1
    return used, have[0] if have else 0


@pytest.mark.parametrize("k", [23, 28, 32, 40, 46, 48, 51, 63, 64])
def test_batch_code_stays_in_its_tile(tmp_path, k):
    p = xg.Program(ldl_solve(k))
    src = plan_probe.batch_source([p], str(tmp_path / "b.hip"))
    used, have = accesses(src, 8)
    assert used + 64 * 8 <= have
    assert have == p.info(0)["n_ws_slots"] * 64 * 8


@pytest.mark.parametrize("keys", [("mpc",), ("quad", "ldl22"), ("rdag1e4",)])
def test_batch_workspace_is_the_plans(tmp_path, keys):
    for key in keys:
        p = xg.Program(configs.program_path(key))
        used, have = accesses(plan_probe.batch_source([p], str(tmp_path / "b.hip")), 4 if p.dtype == "f32" else 8)
        assert have == p.info(0)["n_ws_slots"] * 64 * (4 if p.dtype == "f32" else 8)
        assert used < max(have, 1)
