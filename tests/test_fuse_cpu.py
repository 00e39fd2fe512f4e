"""The graph passes that run before planning, checked on the CPU
(tests/native/fuse_eval.cpp walks the graphs): folding negations keeps every
bit (signs of zeros included), joining products to sums is a fused rounding
per joined sum and removes operations."""

import os
import subprocess

import numpy as np
import pytest

import paper_2408_09662_amd as xg
from tests import parity
from workloads import configs
from workloads.tracer import Graph

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    exe = tmp_path_factory.mktemp("fuse") / "fuse_eval"
    libdir = os.path.dirname(xg._abi.LIB_PATH)
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(libdir, "csrc"), os.path.join(ROOT, "tests", "native", "fuse_eval.cpp"),
                    "-o", str(exe), "-L", libdir, "-l:libxg.so", f"-Wl,-rpath,{libdir}"], check=True)
    return exe


def walk(exe, d, xs, tmp_path):
    desc, inp, outp = tmp_path / "d.txt", tmp_path / "in.bin", tmp_path / "out.bin"
    with open(desc, "w") as f:
        f.write(f"64 {d['n_work']} {len(d['nnz_in'])} " + " ".join(map(str, d["nnz_in"]))
                + f" {len(d['nnz_out'])} " + " ".join(map(str, d["nnz_out"]))
                + f" {len(d['consts'])} " + " ".join(float(c).hex() for c in d["consts"]) + f" {len(d['instr'])}\n")
        for op, o, a, b in d["instr"]:
            f.write(f"{op} {o} {a} {b} 0\n")
    n = xs[0].shape[1]
    with open(inp, "wb") as f:
        f.write(np.int64(n).tobytes())
        f.write(np.ascontiguousarray(np.concatenate(xs, axis=0).T).tobytes())
    subprocess.run([str(exe), str(desc), str(inp), str(outp)], check=True)
    raw = np.fromfile(outp, dtype=np.float64)
    return raw[:-3].reshape(n, 3, sum(d["nnz_out"])), raw[-3:]


@pytest.mark.parametrize("key", ["pend7", "mpc", "quad", "rdag200", "ldl22"])
def test_passes_keep_the_values(driver, tmp_path, key):
    d = xg.load_program_file(configs.program_path(key))
    xs = configs.item_inputs(key, 24)
    y, ops = walk(driver, d, xs, tmp_path)
    assert np.array_equal(y[:, 0].view(np.int64), y[:, 1].view(np.int64))
    tol = parity.TOL_F64_MPC if key == "mpc" else parity.TOL_F64
    assert parity.max_err([y[:, 2].T], [y[:, 0].T]) <= tol
    assert ops[1] <= ops[0] and ops[2] < ops[1]


def test_signs_of_zeros_and_every_sum_form(driver, tmp_path):
    """Each way a negation can meet a product, quotient, sum or difference, at
    zeros of both signs, and each form of fused sum at values whose products
    are exact (one rounding there is the plain result)."""
    g = Graph("forms", "f64")
    a, b, c = g.input(3)
    na, nb = -a, -b
    outs = [na + nb, na - nb, a - nb, na + b, a + nb, na - b, na * b, na * nb, na / (c + 2.0), -(na * nb), na + na,
            a * b + c, a * b - c, c - a * b, a * a + c, (a + a) + c, c - (b + b), na * b + c, c - na * nb,
            a * b + b * c, a * b - b * c, abs_(g, na) + a * c]
    p = g.program([outs])
    d = xg._from_workload(p)
    v = np.array([0.0, -0.0, 1.0, -1.0, 0.5, -3.0])
    xs = [np.array(np.meshgrid(v, v, v)).reshape(3, -1)]
    y, _ = walk(driver, d, xs, tmp_path)
    assert np.array_equal(y[:, 0].view(np.int64), y[:, 1].view(np.int64))
    assert np.array_equal(y[:, 0], y[:, 2])  # (a fused sum may give the other zero)


def abs_(g, x):
    from workloads.tracer import fabs
    return fabs(x)
