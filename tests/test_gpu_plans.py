"""The library's own plans by instance count: the plan for few tiles and the
one that fills the chip give the same bits (sums take their products in the
graph, not in a plan), and match the oracle."""

import numpy as np
import pytest

from oracle.pyoracle import Program as OProg
from tests import parity
from workloads import configs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("key,ns", [("rdag200", (1, 65, 1000)), ("pend7", (63, 1000)), ("pend7_f32", (129,)),
                                    ("ldl22", (64, 777)), ("quad", (65,))])
def test_plans_give_the_same_bits(key, ns):
    import paper_2408_09662_amd as xg
    path = configs.program_path(key)
    lib = xg.Program(path)
    one = xg.Program(path, reg_budget=112)  # one wave per tile at every count
    o = OProg(path)
    for n in ns:
        xs = configs.ITEMS[key].make_inputs(n)
        if lib.dtype == "f32":
            xs = [x.astype(np.float32).astype(np.float64) for x in xs]
        x = [torch.from_numpy(t).to(lib.torch_dtype).cuda() for t in xs]
        print(f"plans: {key} n={n}", flush=True)
        a, b = lib.eval(x), one.eval(x)
        torch.cuda.synchronize()
        assert all(torch.equal(p, q) for p, q in zip(a, b)), (key, n)
        tol = parity.f32_tol(o, xs) if lib.dtype == "f32" else parity.TOL_F64
        assert parity.max_err([t.double().cpu().numpy() for t in a], o.evaluate(xs, 64, threads=8)) <= tol, (key, n)


@pytest.mark.parametrize("key,most,n", [("ldl22", 20000, 16384), ("quad", 20000, 1000)])
def test_workspace_of_a_larger_count_serves_a_smaller(key, most, n):
    """A workspace sized for `most` instances is enough for fewer, whichever
    plan runs them."""
    import paper_2408_09662_amd as xg
    p = xg.Program(configs.program_path(key))
    assert p.workspace_bytes(most) >= p.workspace_bytes(n)
    x = [torch.from_numpy(t).cuda() for t in configs.ITEMS[key].make_inputs(n)]
    ws = torch.empty(max(p.workspace_bytes(most), 8), dtype=torch.uint8, device="cuda")
    assert torch.equal(p.eval(x, workspace=ws)[0], p.eval(x)[0])


@pytest.mark.parametrize("key,n", [("mpc", 65), ("ldl48", 130)])
def test_plans_ranked_by_transfers(key, n):
    """Programs that spill to the workspace: their plan for few tiles against
    one wave per tile, bit by bit, and the oracle."""
    import paper_2408_09662_amd as xg
    path = configs.program_path(key)
    xs = configs.ITEMS[key].make_inputs(n)
    x = [torch.from_numpy(t).cuda() for t in xs]
    a, b = xg.Program(path).eval(x), xg.Program(path, reg_budget=112).eval(x)
    torch.cuda.synchronize()
    assert all(torch.equal(p, q) for p, q in zip(a, b)), key
    ref = OProg(path).evaluate(xs, 64, threads=8)
    assert parity.max_err([t.cpu().numpy() for t in a], ref) <= parity.TOL_F64, key
