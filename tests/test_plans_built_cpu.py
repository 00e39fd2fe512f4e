"""What compiling ahead covers: the code of both of a mode's plans, and a plan
for few tiles that cannot be built leaves the other to run every count."""

import pytest

import paper_2408_09662_amd as xg
from tests import plan_probe
from workloads import configs


@pytest.mark.parametrize("mode", [0, 2])
def test_precompile_builds_both_plans(mode):
    from workloads.pendulum import pendulum
    p = xg.Program(configs.program_path("rdag200") if mode == 0 else pendulum(4))
    p.precompile(mode)
    assert plan_probe.compiled(p, mode, False)
    assert plan_probe.compiled(p, mode, True) == plan_probe.few(p, mode, 1)
    assert mode != 0 or plan_probe.few(p, mode, 1)


def test_both_plans_compile_once(tmp_path, monkeypatch):
    """Without the on-disk cache too: the code compiled is the code kept."""
    monkeypatch.setenv("XG_NO_CACHE", "1")
    monkeypatch.setenv("XG_CACHE_DIR", str(tmp_path))
    monkeypatch.setenv("XG_DUMP_DIR", str(tmp_path))
    p = xg.Program(configs.program_path("rdag200"))
    p.precompile(0)
    first = {f: f.stat().st_mtime_ns for f in tmp_path.glob("*.co")}
    assert len(first) == 2
    with pytest.raises(xg.XgError, match="DEVICE"):
        p.compile(0)
    assert {f: f.stat().st_mtime_ns for f in tmp_path.glob("*.co")} == first


def test_plan_for_few_tiles_that_does_not_build():
    p = xg.Program(configs.program_path("rdag200"))
    assert plan_probe.few(p, 0, 1000)
    plan_probe.spoil_few(p, 0)
    p.precompile(0)
    assert plan_probe.compiled(p, 0, False)
    assert not plan_probe.few(p, 0, 1000)
