"""Both sides of the count where a mode's plan changes: which plan runs, the
same bits per instance, and nothing stored past a workspace of exactly the size
asked for."""

import pytest

from tests import plan_probe
from workloads import configs
from workloads.pendulum import pendulum

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GUARD = 1 << 16


def guarded(p, n, mode):
    nb = p.workspace_bytes(n, mode)
    return nb, torch.full((nb + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")


def last_few(p, mode):
    """The largest count that runs the plan for few tiles."""
    return max(n for n in range(64, 262144 + 65, 64) if plan_probe.few(p, mode, n))


@pytest.mark.parametrize("key", ["rdag200", "ldl22", "pend7_f32"])
def test_forward_across_the_switch(key):
    import paper_2408_09662_amd as xg
    p = xg.Program(configs.program_path(key))
    n = last_few(p, 0)
    assert plan_probe.few(p, 0, n) and not plan_probe.few(p, 0, n + 1)
    x = [torch.from_numpy(t).to(p.torch_dtype).cuda() for t in configs.ITEMS[key].make_inputs(n + 1)]
    got = {}
    for m in (n, n + 1, n - 1):
        nb, ws = guarded(p, m, 0)
        print(f"switch: {key} n={m}", flush=True)
        got[m] = p.eval([t[:, :m] for t in x], n=m, workspace=ws)
        torch.cuda.synchronize()
        assert bool((ws[nb:] == 0xA5).all())
    for a, b, c in zip(got[n], got[n + 1], got[n - 1]):
        assert torch.equal(a, b[:, :n]) and torch.equal(a[:, :n - 1], c)


@pytest.mark.parametrize("links", [4, 6])
@pytest.mark.parametrize("mode", [1, 2])
def test_adjoint_across_the_switch(mode, links):
    import paper_2408_09662_amd as xg
    p = xg.Program(pendulum(links))
    n = 64 * 256
    assert plan_probe.few(p, mode, n) and not plan_probe.few(p, mode, n + 1)
    g = torch.Generator(device="cuda").manual_seed(links)
    x, s = (torch.randn((2 * links, n + 1), generator=g, dtype=torch.float64, device="cuda") for _ in range(2))
    got = {}
    for m in (n, n + 1):
        nb, ws = guarded(p, m, mode)
        print(f"switch: pendulum {links} mode {mode} n={m}", flush=True)
        r = p.eval_adjoint([x[:, :m]], [s[:, :m]], with_outputs=mode == 2, n=m, workspace=ws)
        torch.cuda.synchronize()
        assert bool((ws[nb:] == 0xA5).all())
        got[m] = r[0] + r[1] if mode == 2 else r
    for a, b in zip(got[n], got[n + 1]):
        assert torch.equal(a, b[:, :n])
