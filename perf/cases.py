"""Performance cases: what programs built on this library have it do.

A case names a path (one plain eval call, a forward evaluation bound to fixed
buffers, a gradient through autograd, the fused forward + adjoint call, a
graph-captured closed-loop rollout, one persistent launch of several
programs), a program of the repository's workload families, an element type and an instance count.  Programs are
loaded with the library's default options, as a first user of a program does;
only the case that says "tuned" asks the autotuner for its plan, as the
repository's benchmark does.  A loaded program is kept for the process, like
the plan of any long-running simulation or controller.
"""

import functools
import math

import torch

import paper_2408_09662_amd as xg
from workloads import ldl, mpc, pendulum, quadcopter, rdag


def listed():
    return [
        # the smallest call: a 200-operation expression for 1,000 instances,
        # outputs allocated by the call; latency and launch decide it
        dict(name="dag200_f64_1000", path="call", program="rdag", size=200, seed=1, dtype="f64", n=1000),
        # a simulation step of a 7-link pendulum for the environments of one
        # training job, with the plan its owner had tuned
        dict(name="pend7_f64_16384_tuned", path="tuned", program="pendulum", size=7, dtype="f64", n=16384),
        # the same step for a few thousand environments, an odd count, as loaded
        dict(name="pend7_f64_4097", path="forward", program="pendulum", size=7, dtype="f64", n=4097),
        # and for a large batch of samples (every SIMD has work)
        dict(name="pend7_f64_65536", path="forward", program="pendulum", size=7, dtype="f64", n=65536),
        # single precision, as most learning code runs it
        dict(name="pend7_f32_16384", path="forward", program="pendulum", size=7, dtype="f32", n=16384),
        # gradient of the squared final state through torch.autograd
        dict(name="pend7_grad_f64_65536", path="grad", program="pendulum", size=7, dtype="f64", n=65536),
        # value and gradient in one call, single precision, a ragged batch
        dict(name="pend7_fused_f32_8191", path="fused", program="pendulum", size=7, dtype="f32", n=8191),
        # closed-form MPC for the environments of a training job
        dict(name="mpc3_f64_4096", path="forward", program="mpc", size=3, dtype="f64", n=4096),
        # the same controller over a large set of sampled states
        dict(name="mpc3_f64_65536", path="forward", program="mpc", size=3, dtype="f64", n=65536),
        # 20 closed-loop steps of 10,000 quadcopters from one captured graph
        dict(name="quad_rollout_10000x20", path="rollout", program="quad", size=20, dtype="f64", n=10000),
        # LDL^T solves of 48 x 48 systems, the larger end of the solve family
        dict(name="ldl48_f64_10000", path="forward", program="ldl", size=48, dtype="f64", n=10000),
        # programs of uneven size and count in one persistent launch
        dict(name="batch_65536_8192_500", path="batch", program="batch", size=3000, seed=53, dtype="f32", n=65536,
             n2=8192, n3=500),
    ]


def _logn(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n))


def draw(rng):
    path = rng.choice(["forward"] * 5 + ["call", "grad", "fused", "fused", "rollout", "batch"])
    if path == "rollout":
        return dict(path=path, program="quad", size=rng.randint(5, 20), dtype="f64", n=_logn(rng, 64, 10000))
    if path == "batch":
        return dict(path=path, program="batch", size=rng.randint(1000, 3000), seed=rng.randint(1, 1000), dtype="f32",
                    n=_logn(rng, 4096, 65536), n2=_logn(rng, 256, 8192), n3=_logn(rng, 64, 512))
    if path in ("grad", "fused"):
        return dict(path=path, program="pendulum", size=rng.randint(2, 7), dtype=rng.choice(["f64", "f64", "f32"]),
                    n=_logn(rng, 64, 65536))
    prog = rng.choice(["pendulum", "pendulum", "mpc", "mpc", "ldl", "rdag"])
    c = dict(path=path, program=prog)
    if prog == "pendulum":
        c.update(size=rng.randint(2, 7), dtype=rng.choice(["f64", "f64", "f32"]), n=_logn(rng, 64, 65536))
    elif prog == "mpc":
        c.update(size=rng.randint(1, 3), dtype=rng.choice(["f64", "f64", "mixed"]), n=_logn(rng, 64, 65536))
    elif prog == "ldl":
        k = _logn(rng, 4, 48)
        c.update(size=k, dtype="f64", n=_logn(rng, 64, 100000 if k <= 22 else 10000))
    else:
        c.update(size=rng.randint(100, 1000), seed=rng.randint(1, 1000), dtype=rng.choice(["f64", "f32"]),
                 n=_logn(rng, 64, 65536))
    return c


# ------------------------------------------------------------------ programs
@functools.lru_cache(maxsize=None)
def _source(program, size, dtype, seed):
    """The workload's instruction list (what a symbolic front end hands over)."""
    if program == "rdag":
        return rdag.rdag(seed, 16 if size >= 1000 else 8, size, dtype=dtype)
    if program == "pendulum":
        return pendulum.pendulum(size, dtype=dtype)
    if program == "mpc":
        return mpc.cartpole_mpc(iters=size, **({"precision": "mixed"} if dtype == "mixed" else {}))
    if program == "ldl":
        return ldl.ldl_solve(size)
    return quadcopter.quad_closed_loop()


def _sources(case):
    if case["path"] == "batch":  # a DAG for many instances, solves for some, a large DAG for few
        return [_source("rdag", 1000, "f32", 51), _source("ldl", 22, "f64", 0),
                _source("rdag", case["size"], "f32", case["seed"])]
    return [_source(case["program"], case["size"], case["dtype"], case.get("seed", 0))]


def _counts(case):
    return [case["n"], case["n2"], case["n3"]] if case["path"] == "batch" else [case["n"]]


_kept = {}


def _loaded(case):
    """The program (or batch) the case's owner keeps loaded."""
    key = tuple(sorted((k, v) for k, v in case.items() if k not in ("name", "n", "n2", "n3")))
    if case["path"] == "tuned":
        key += (case["n"],)
    if key not in _kept:
        ps = [xg.Program(s) for s in _sources(case)]
        _kept[key] = (ps, xg.Batch(ps)) if case["path"] == "batch" else (ps, None)
    return _kept[key]


# -------------------------------------------------------------------- inputs
def _inputs(case, seed):
    """Per program: its input tensors, drawn from the workload's distributions."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def u(k, n, lo, hi):
        return lo + (hi - lo) * torch.rand((k, n), generator=g, dtype=torch.float64, device="cuda")

    def normal(k, n):
        return torch.randn((k, n), generator=g, dtype=torch.float64, device="cuda")

    def spd(k, n):  # strictly diagonally dominant, packed lower triangle
        a = u(k * (k + 1) // 2, n, -1.0, 1.0)
        rows = torch.tensor([ldl.tri_index(i, i) for i in range(k)], device="cuda")
        a[rows] = k + u(k, n, 0.0, 1.0)
        return [a, normal(k, n)]

    def one(src, program, size, n):
        if program == "rdag":
            x = [u(src.nnz_in[0], n, -1.0, 1.0)]
        elif program == "pendulum":
            x = [torch.cat([u(size, n, -math.pi, math.pi), normal(size, n)])]
        elif program == "mpc":
            scale = torch.tensor([[1.0], [math.pi], [1.0], [1.0]], dtype=torch.float64, device="cuda")
            x = [(u(4, n, -1.0, 1.0) * scale).contiguous()]
        elif program == "ldl":
            x = spd(size, n)
        else:
            z = torch.zeros((6, n), dtype=torch.float64, device="cuda")
            z[3:5] = u(2, n, -3.0, 3.0)
            z[5] = u(1, n, -6.0, 6.0)[0]
            m = u(1, n, 0.8, 1.2)
            x = [z, torch.cat([m, u(1, n, 0.008, 0.012), u(1, n, 0.1, 0.2), u(1, n, 0.75, 1.5) * m * 9.81,
                               u(3, n, 1.0, 10.0), u(3, n, 0.1, 1.0), u(2, n, 0.1, 1.0)])]
        return [t.to(torch.float32) if src.dtype == "f32" else t for t in x]

    srcs, ns = _sources(case), _counts(case)
    if case["path"] == "batch":
        return [one(srcs[0], "rdag", 0, ns[0]), one(srcs[1], "ldl", 22, ns[1]), one(srcs[2], "rdag", 0, ns[2])]
    x = one(srcs[0], case["program"], case["size"], ns[0])
    if case["path"] == "fused":  # the seeds of a loss's gradient with respect to the outputs
        x.append(normal(srcs[0].nnz_out[0], ns[0]).to(x[0].dtype))
    return [x]


# ---------------------------------------------------------------- one pass
def prepare(case, seed):
    ps, batch = _loaded(case)
    xs = _inputs(case, seed)
    st = {"path": case["path"], "p": ps[0], "x": xs[0]}
    if case["path"] in ("forward", "tuned"):
        if case["path"] == "tuned" and not st["p"].__dict__.get("was_tuned", False):
            xg.autotune(st["p"], xs[0])
            st["p"].was_tuned = True
        st["out"] = st["p"].alloc_outputs(case["n"])
        st["call"] = st["p"].bind_eval(xs[0], st["out"])
    elif case["path"] == "fused":
        st["grads"] = [torch.empty_like(xs[0][0])]
        st["out"] = st["p"].alloc_outputs(case["n"])
    elif case["path"] == "batch":
        st.update(b=batch, xs=xs, out=[p.alloc_outputs(n) for p, n in zip(ps, _counts(case))],
                  ws=batch.workspace(_counts(case)))
    elif case["path"] == "rollout":
        z, th = xs[0]
        st["s"] = [torch.empty_like(z), torch.empty_like(z)]
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            st["graph"] = xg.capture_rollout(st["p"], st["s"][0], st["s"][1], [th], case["size"], stream=side)
        torch.cuda.current_stream().wait_stream(side)
        st["end"] = st["s"][case["size"] % 2]
    return st


def run(state):
    path, p, x = state["path"], state["p"], state["x"]
    if path == "call":
        return p.eval(x)
    if path in ("forward", "tuned"):
        state["call"]()
        return state["out"]
    if path == "grad":
        xr = x[0].detach().requires_grad_(True)
        y = xg.XgFunction.apply(p, xr)
        (gx,) = torch.autograd.grad((y * y).sum(), xr)
        return [y.detach(), gx]
    if path == "fused":
        g, y = p.eval_adjoint(x[:1], x[1:], grads=state["grads"], outputs=state["out"], with_outputs=True)
        return [y, g]
    if path == "batch":
        return state["b"].eval(state["xs"], state["out"], workspace=state["ws"])
    state["s"][0].copy_(x[0])  # every environment starts its episode
    state["graph"].launch()
    return state["end"]


# ------------------------------------------------------------------- amounts
def work(case):
    nbytes = flops = 0
    for s, n in zip(_sources(case), _counts(case)):
        es = 4 if s.dtype == "f32" else 8
        ops = s.n_arith()
        io = sum(s.nnz_in) + sum(s.nnz_out)
        if case["path"] in ("grad", "fused"):  # value and gradient: inputs, seeds, outputs, gradients
            ops, io = 3 * ops, 2 * io
        if case["path"] == "rollout":
            ops *= case["size"]
        nbytes += es * io * n
        flops += ops * n
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------- the same in 64 bits
def _walk(src, x, keep):
    """The instruction list walked in torch, binary64 (`keep`: for autograd)."""
    c = [float(v) for v in src.consts]
    w, y = {}, [[None] * k for k in src.nnz_out]
    zero = torch.zeros_like(x[0][0])
    unary = {"SQRT": torch.sqrt, "EXP": torch.exp, "LOG": torch.log, "SIN": torch.sin, "COS": torch.cos,
             "TAN": torch.tan, "TANH": torch.tanh, "ATAN": torch.atan, "FABS": torch.abs, "NEG": torch.neg,
             "SQ": lambda a: a * a, "ASSIGN": lambda a: a}
    binary = {"ADD": torch.add, "SUB": torch.sub, "MUL": torch.mul, "DIV": torch.div, "FMIN": torch.fmin,
              "FMAX": torch.fmax, "POW": torch.pow, "ATAN2": torch.atan2,
              "LT": lambda a, b: (a < b).to(zero.dtype), "LE": lambda a, b: (a <= b).to(zero.dtype)}
    with torch.set_grad_enabled(keep):
        for op, o, a, b in src.instrs:
            if op == "INPUT":
                w[o] = x[a][b]
            elif op == "CONST":
                w[o] = zero + c[a]
            elif op == "OUTPUT":
                y[o][b if b >= 0 else 0] = w[a]
            elif op in unary:
                w[o] = unary[op](w[a])
            else:
                w[o] = binary[op](w[a], w[b])
        return [torch.stack(list(v)) for v in y]


def exact(case, seed):
    xs = [[t.double() for t in x] for x in _inputs(case, seed)]
    srcs = _sources(case)
    if case["path"] == "batch":
        return [_walk(s, x, False) for s, x in zip(srcs, xs)]
    src, x = srcs[0], xs[0]
    if case["path"] == "rollout":
        z = x[0]
        for _ in range(case["size"]):
            z = _walk(src, [z, x[1]], False)[0]
        return z
    if case["path"] in ("grad", "fused"):
        rows = [r.clone().requires_grad_(True) for r in x[0]]
        y = _walk(src, [rows], True)[0]
        seeds = 2.0 * y.detach() if case["path"] == "grad" else x[1]
        g = torch.stack(torch.autograd.grad(y, rows, seeds))
        return [y.detach(), g] if case["path"] == "grad" else [[y.detach()], [g]]
    return _walk(src, x, False)
