"""Planning a wide program: each choice of the phased scheduler looks at what
changed, not at every ready cluster."""

import resource

import paper_2408_09662_amd as xg
from tests import plan_probe
from workloads.rdag import rdag


def test_wide_program_plans_quickly():
    """A 30,000-operation DAG on 64 inputs: processor time, which does not
    depend on what else runs (about 15 s; 240 with a scan per choice)."""
    p = xg.Program(rdag(9, 64, 30000, dtype="f32"))
    t = resource.getrusage(resource.RUSAGE_SELF).ru_utime
    code, phases = plan_probe.code(p, 0, 64)
    assert code and phases > 1
    assert resource.getrusage(resource.RUSAGE_SELF).ru_utime - t < 60
