"""Batches of default-loaded programs whose plans are made with less than the
program's register budget: results bit by bit as alone, against the oracle,
and nothing stored past the workspace."""

import numpy as np
import pytest

from oracle.pyoracle import Program as OProg
from tests import parity
from workloads import ldl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def test_spilling_solve_in_a_batch(tmp_path):
    import paper_2408_09662_amd as xg
    srcs = [ldl.ldl_solve(46), ldl.ldl_solve(22)]
    ps = [xg.Program(s) for s in srcs]
    b = xg.Batch(ps)
    ns = [130, 65]
    host = [ldl.spd_inputs(17, s.nnz_in[1], n) for s, n in zip(srcs, ns)]
    xs = [[torch.from_numpy(x).cuda() for x in h] for h in host]
    outs = [p.alloc_outputs(n) for p, n in zip(ps, ns)]
    nb, guard = b.workspace_bytes(ns), 1 << 16
    ws = torch.full((nb + guard,), 0xA5, dtype=torch.uint8, device="cuda")
    print("batch of 46 x 46 and 22 x 22 solves", flush=True)
    b.eval(xs, outs, workspace=ws)
    alone = [p.eval(x) for p, x in zip(ps, xs)]
    torch.cuda.synchronize()
    assert bool((ws[nb:] == 0xA5).all())
    for k, s in enumerate(srcs):
        assert torch.equal(outs[k][0], alone[k][0])
        s.save(str(tmp_path / "p.xgp"))
        ref = OProg(str(tmp_path / "p.xgp")).evaluate(host[k], 64, threads=8)
        assert parity.max_err([outs[k][0].cpu().numpy()], ref) <= parity.TOL_F64
