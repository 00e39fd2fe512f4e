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


def test_wide_workgroups_have_the_budgets_of_theirs():
    """The library's budgets are those of one wave on a SIMD: batch candidates
    of more lanes hold fewer values each, and 64 lanes run as loaded."""
    keys, ns = ("rdag1e4", "ldl48"), (512, 4000)
    own = {b: [xg.Program(configs.program_path(k), **o) for k, o in zip(keys, os)] for b, os in
           ((512, (dict(reg_budget=200, lds_slots=638), dict(reg_budget=112, lds_slots=319))),
            (1024, (dict(reg_budget=96, lds_slots=638), dict(reg_budget=48, lds_slots=319))))}
    a = plan_probe.batch_candidates([xg.Program(configs.program_path(k)) for k in keys], ns)
    b, c = (plan_probe.batch_candidates(own[w], ns) for w in (512, 1024))
    assert sorted(a) == [64, 256, 512, 1024]
    assert a[256] == b[256] and a[512] == b[512] and a[1024] == c[1024]
    assert a[64] != b[64]


def test_64_lanes_run_as_loaded(tmp_path):
    ps = [xg.Program(configs.program_path(k)) for k in ("rdag1e3", "ldl48")]
    src = plan_probe.batch_source(ps, str(tmp_path / "b.hip"))
    h = 1469598103934665603
    for c in src.encode():
        h = (h ^ c) * 1099511628211 & (1 << 64) - 1
    assert plan_probe.batch_candidates(ps, (65536, 4000))[64] == h


@pytest.mark.parametrize("tiles,cost,grid", [
    ([1024, 128, 8, 32], [1500, 15000, 150000, 50000], 256),  # the 8 long tiles bound the launch
    ([1024, 128, 8], [1500, 5000, 4500], 1024),               # the many short ones do
    ([3, 0], [100, 10 ** 9], 3),                              # an empty program's tiles cost nothing
    ([128], [7], 128), ([257], [7], 257), ([5000], [7], 1024),
])
def test_workgroups_of_a_launch(tiles, cost, grid):
    assert plan_probe.batch_grid(tiles, cost, 1024, 256) == grid
    assert plan_probe.batch_grid(tiles, cost, 64, 256) == min(grid, 64)
