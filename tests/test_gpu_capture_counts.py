"""A program evaluated once may be captured at any other count: the code of
the plan that fills the chip is loaded with the plan for few tiles."""

import pytest

from tests import plan_probe
from workloads import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("key,warm,n", [("rdag200", 100, 300000), ("rdag200", 300000, 100), ("ldl22", 64, 40000)])
def test_capture_after_another_count(key, warm, n):
    import paper_2408_09662_amd as xg
    p = xg.Program(configs.program_path(key))
    p.eval([torch.from_numpy(t).cuda() for t in configs.ITEMS[key].make_inputs(warm)])
    assert plan_probe.few(p, 0, warm) != plan_probe.few(p, 0, n)
    assert plan_probe.loaded(p, 0, False) == 1
    x = [torch.from_numpy(t).cuda() for t in configs.ITEMS[key].make_inputs(n)]
    out = p.alloc_outputs(n)
    torch.cuda.synchronize()
    print(f"capture {key} n={n} after n={warm}", flush=True)
    before = plan_probe.loaded(p, 0, True)
    g = torch.cuda.CUDAGraph()
    ws = p.workspace(n)
    with torch.cuda.graph(g):
        p.eval(x, out, workspace=ws)
    assert plan_probe.loaded(p, 0, True) == before
    ref = p.eval(x)
    for k in range(3):
        for o in out:
            o.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref)), k
