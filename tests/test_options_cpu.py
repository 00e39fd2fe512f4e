"""What one launch option set changes in the plans of a program whose other
options are the library's."""

import pytest

import paper_2408_09662_amd as xg
from tests import plan_probe
from workloads import configs
from workloads.pendulum import pendulum


def code(p, mode):
    return p.info(mode)["code_hash"]


@pytest.mark.parametrize("opt", [dict(block=64), dict(ipt=1), dict(waves=1), dict(prefetch=24), dict(chunk_ops=20000)])
def test_defaults_written_out(opt):
    src = pendulum(5)
    a, b = xg.Program(src), xg.Program(src, **opt)
    for mode in (0, 1, 2):
        assert code(a, mode) == code(b, mode)
        for n in (64, 16384, 65536):
            assert plan_probe.few(a, mode, n) == plan_probe.few(b, mode, n)
    assert plan_probe.few(b, 0, 64)


@pytest.mark.parametrize("links,dtype", [(3, "f64"), (4, "f64"), (5, "f64"), (4, "f32")])
@pytest.mark.parametrize("opt", [dict(prefetch=48), dict(chunk_ops=5000)])
def test_adjoint_budgets_beside_another_option(links, dtype, opt):
    """The adjoint then has the budgets of a program that sets options: those
    the library's own long and short kernels take are not for other chunks."""
    src = pendulum(links, dtype=dtype)
    given = dict(reg_budget=112, lds_slots=319) if dtype == "f64" else dict(reg_budget=200, lds_slots=638)
    for mode in (1, 2):
        assert code(xg.Program(src, **opt), mode) == code(xg.Program(src, **opt, **given), mode)


def test_forward_budgets_beside_another_option():
    """The forward keeps the library's, lowered for a program that overflows
    any budget by far."""
    src = configs.program_path("ldl48")
    a, b = xg.Program(src, prefetch=48), xg.Program(src, prefetch=48, reg_budget=160, lds_slots=79)
    assert code(a, 0) == code(b, 0)
    assert a.info(0)["n_ws_slots"] == b.info(0)["n_ws_slots"]
