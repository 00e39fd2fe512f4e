"""Programs with binary32 tags: their phased tiles keep few values beyond the
registers and the LDS (workspace slots per instance, spills)."""

import pytest

import paper_2408_09662_amd as xg
from workloads import configs


@pytest.mark.parametrize("lds,slots", [(34, 799), (159, 638)])
def test_two_wave_tiles_of_the_mixed_mpc(lds, slots):
    p = xg.Program(configs.program_path("mpc_mixed"), waves=2, coop_phase=300, reg_budget=168, lds_slots=lds)
    i = p.info(0)
    assert i["n_ws_slots"] <= slots and i["n_spills"] <= 2524
