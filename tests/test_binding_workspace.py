"""The binding's workspaces follow the program's current plan: tuning, also
through the C entry points or on another thread, changes what an evaluation
needs (the library and torch are stood in for; no GPU)."""

import threading
import types

import pytest

import paper_2408_09662_amd as xg
from workloads import configs


class Buffer:
    def __init__(self, nb):
        self.nb = nb

    def numel(self):
        return self.nb

    def data_ptr(self):
        return 4096


@pytest.fixture
def prog(monkeypatch):
    p = xg.Program(configs.program_path("rdag200"))
    cuda = types.SimpleNamespace(current_device=lambda: 0)
    torch = types.SimpleNamespace(empty=lambda nb, **k: Buffer(nb), uint8=None, cuda=cuda, float64=None)
    monkeypatch.setattr(xg, "_torch", lambda: torch)
    return p


def test_size_is_the_current_plans(prog, monkeypatch):
    need = {"bytes": 512}
    monkeypatch.setattr(prog, "workspace_bytes", lambda n, mode=0: need["bytes"])
    assert prog.workspace(1000).numel() == 512
    need["bytes"] = 8192  # a plan with more spills
    assert prog.workspace(1000).numel() >= 8192


def test_eval_after_a_plan_that_needed_none(prog, monkeypatch):
    need = {"bytes": 0}
    calls = []

    def xg_eval(h, n, pi, li, po, lo, ws, stream):
        calls.append(ws)
        return 0 if ws or not need["bytes"] else 1

    monkeypatch.setattr(prog, "workspace_bytes", lambda n, mode=0: need["bytes"])
    monkeypatch.setattr(xg, "lib", lambda: types.SimpleNamespace(xg_eval=xg_eval))
    monkeypatch.setattr(xg, "_ptrs", lambda *a: (None, None))
    monkeypatch.setattr(xg, "_stream_handle", lambda s: None)
    for _ in range(2):
        prog.eval([None], [None], n=1000)
    need["bytes"] = 4096
    prog.eval([None], [None], n=1000)
    prog.eval([None], [None], n=1000)
    assert calls == [None, None, None, 4096, 4096]


def test_a_refused_call_raises(prog, monkeypatch):
    monkeypatch.setattr(prog, "workspace_bytes", lambda n, mode=0: 0)
    monkeypatch.setattr(xg, "lib", lambda: types.SimpleNamespace(xg_eval=lambda *a: 1))
    monkeypatch.setattr(xg, "_ptrs", lambda *a: (None, None))
    monkeypatch.setattr(xg, "_stream_handle", lambda s: None)
    for _ in range(2):
        with pytest.raises(xg.XgError):
            prog.eval([None], [None], n=1000)


def test_many_counts_on_many_threads(prog, monkeypatch):
    import sys
    monkeypatch.setattr(prog, "workspace_bytes", lambda n, mode=0: 8 * n)
    errors = []

    def work(k):
        try:
            for n in range(k, 40000, 8):
                assert prog.workspace(n).numel() >= 8 * n
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    old = sys.getswitchinterval()
    sys.setswitchinterval(1e-6)
    try:
        ts = [threading.Thread(target=work, args=(k + 1,)) for k in range(8)]
        for t in ts:
            t.start()
        for t in ts:
            t.join()
    finally:
        sys.setswitchinterval(old)
    assert not errors
