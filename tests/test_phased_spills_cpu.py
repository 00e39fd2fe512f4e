"""Phased tiles set by the caller, for programs that spill to the workspace:
the plan is the one with the cheaper spills."""

import pytest

import paper_2408_09662_amd as xg
from workloads import configs


@pytest.mark.parametrize("key,waves,lds,slots", [("ldl48", 2, 159, 2014), ("ldl48", 4, 79, 2639),
                                                 ("mpc", 4, 79, 1524), ("mpc_m1", 2, 159, 237)])
def test_workspace_of_phased_tiles(key, waves, lds, slots):
    p = xg.Program(configs.program_path(key), waves=waves, coop_phase=300, reg_budget=168, lds_slots=lds)
    assert p.info(0)["n_ws_slots"] <= slots
