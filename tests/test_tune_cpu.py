"""Tuning starts from what runs untuned: the candidates hold the very plans of
the program as loaded, so tuning never ends on a slower one."""

import pytest

import paper_2408_09662_amd as xg
from tests import plan_probe
from workloads import configs
from workloads.pendulum import pendulum


@pytest.mark.parametrize("key,ns", [("ldl48", (1000, 65536)), ("mpc", (4096, 200000)), ("quad", (10000,)),
                                    ("rdag200", (1000, 100000)), ("pend7", (16384, 65536)), ("rdag1e4", (8192,))])
def test_candidates_hold_the_loaded_plans(key, ns):
    p = xg.Program(configs.program_path(key))
    for n in ns:
        runs = plan_probe.code(p, 0, n)[0]
        assert runs in [h for h, library in plan_probe.candidates(p, 0, n) if library]


@pytest.mark.parametrize("links,dtype,ns", [(4, "f64", (1000, 65536)), (6, "f64", (1000, 65536)), (4, "f32", (1000,))])
@pytest.mark.parametrize("mode", [1, 2])
def test_adjoint_candidates_hold_the_loaded_plans(mode, links, dtype, ns):
    p = xg.Program(pendulum(links, dtype=dtype))
    for n in ns:
        runs = plan_probe.code(p, mode, n)[0]
        assert runs in [h for h, library in plan_probe.candidates(p, mode, n) if library]


def test_programs_with_options_have_no_library_candidate():
    p = xg.Program(configs.program_path("rdag200"), reg_budget=100, lds_slots=40)
    assert not any(library for _, library in plan_probe.candidates(p, 0, 1000))


@pytest.mark.parametrize("fanout", [2, 4])
def test_adjoint_candidates_vary_the_fanout(fanout):
    """Short leaves with either fan-out: which is faster depends on the count."""
    src = pendulum(4)
    p = xg.Program(src, reg_budget=149, adj_seg_ops=150, adj_fanout=fanout, lds_slots=319)
    assert plan_probe.code(p, 2, 16384)[0] in [h for h, _ in plan_probe.candidates(xg.Program(src), 2, 16384)]
