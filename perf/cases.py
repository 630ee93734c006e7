"""Timing cases of the library: what users of the package run, through its
public entry points.

Every case is a dict: `op` names the entry point, the other values are its
sizes and options.

  gram            packed lower triangle of A^t A (paper_1902_02104_amd.gram)
  gram_rows       packed lower triangle of A A^t
  cholesky        factor of the packed product, in place on a copy
  cholesky_solve  forward and back substitution with the factor
  atb             A^t B
  normal_solve    least squares through the normal equations
  project         projection onto the columns of A
  serve           a burst of requests through the serving loop

`dtype` is f64, f32, bf16x3 or fp8; the result has the entry point's default
type (float32 for the three forms with float input; asking for a double
result changes the store of C only).  Inputs are made on the device from the
seed: entries of A uniform in [-1, 1] (N(0, 1) for served requests), and
Gram matrices and factors of matrices with twice as many rows as columns.
"""
from __future__ import annotations

import math
import random

import torch

import paper_1902_02104_amd as P
from paper_1902_02104_amd import serving

DTYPES = {"f64": P.F64, "f32": P.F32, "bf16x3": P.F32_BF16X3, "fp8": P.F32_FP8}

# The largest product a case may hold: m n^2 of the 10000 x 10000 square and
# the bytes of the 262144 x 2048 least-squares matrix.
MOST_MN2 = 1.1e12
MOST_BYTES = 262144 * 2048 * 8


def listed():
    return [
        # one small product: the latency of a call (the smoke test's shape)
        {"name": "gram_f64_256x192", "op": "gram", "dtype": "f64", "m": 256, "n": 192, "pad": 0, "depth": -1},
        # an ordinary product with ragged sizes: fewer tiles than the chip has CUs
        {"name": "gram_f64_3001x1203", "op": "gram", "dtype": "f64", "m": 3001, "n": 1203, "pad": 0, "depth": -1},
        # the larger square of the benchmark
        {"name": "gram_f64_10000x10000", "op": "gram", "dtype": "f64", "m": 10000, "n": 10000, "pad": 0,
         "depth": -1},
        # the middle of the serving range (m 1024..65536, n 64..4096), called directly
        {"name": "gram_f32_8192x509", "op": "gram", "dtype": "f32", "m": 8192, "n": 509, "pad": 0, "depth": -1},
        # the companion product of a wide matrix: similarities between its rows
        {"name": "gram_rows_f32_1000x20011", "op": "gram_rows", "dtype": "f32", "m": 1000, "n": 20011, "pad": 0},
        # the precision forms at the benchmark's size
        {"name": "gram_bf16x3_8192x8192", "op": "gram", "dtype": "bf16x3", "m": 8192, "n": 8192, "pad": 0,
         "depth": -1},
        {"name": "gram_fp8_8192x8192", "op": "gram", "dtype": "fp8", "m": 8192, "n": 8192, "pad": 0, "depth": -1},
        # the factor of the benchmark's normal equations and its use for one right-hand side
        {"name": "cholesky_f64_10000", "op": "cholesky", "dtype": "f64", "n": 10000},
        {"name": "cholesky_solve_f64_10000_r1", "op": "cholesky_solve", "dtype": "f64", "n": 10000, "nrhs": 1},
        # the least-squares workload of the benchmark
        {"name": "normal_solve_f64_262144x2048_r1", "op": "normal_solve", "dtype": "f64", "m": 262144, "n": 2048,
         "nrhs": 1},
        # an ordinary projection: short kernels in a chain, a few right-hand sides
        {"name": "project_f32_20011x333_r4", "op": "project", "dtype": "f32", "m": 20011, "n": 333, "nrhs": 4},
        # a burst of requests of the serving stream's shapes, results taken on the device
        {"name": "serve_f32_32", "op": "serve", "dtype": "f32", "count": 32, "shapes": 6},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fits(m, n, dtype):
    return m * n * n <= MOST_MN2 and m * n * (8 if dtype == "f64" else 4) <= MOST_BYTES


def draw(rng):
    op = rng.choices(["gram", "gram_rows", "cholesky", "cholesky_solve", "atb", "normal_solve", "project", "serve"],
                     [10, 2, 3, 3, 1, 2, 2, 1])[0]
    if op == "serve":
        return {"op": op, "dtype": "f32", "count": rng.randint(4, 32), "shapes": rng.randrange(1 << 20)}
    if op in ("cholesky", "cholesky_solve"):
        c = {"op": op, "dtype": rng.choice(["f64", "f64", "f32"]), "n": _log(rng, 24, 10000)}
        if op == "cholesky_solve":
            c["nrhs"] = rng.choice([1, 1, 2, 3, 8, 16, 33])
        return c
    dtype = rng.choice(["f64", "f64", "f32", "f32", "bf16x3", "fp8"] if op in ("gram", "gram_rows") else
                       ["f64", "f32"])
    while True:
        if op == "gram":
            m, n = _log(rng, 16, 262144), _log(rng, 16, 10000)
        elif op == "gram_rows":
            m, n = _log(rng, 16, 8192), _log(rng, 16, 65536)
        else:
            n = _log(rng, 16, 2048)
            m = _log(rng, 2 * n, 262144)
        if _fits(n, m, dtype) if op == "gram_rows" else _fits(m, n, dtype):
            break
    c = {"op": op, "dtype": dtype, "m": m, "n": n}
    if op in ("gram", "gram_rows"):
        c["pad"] = rng.choice([0, 0, 0, 1, 3, 8])  # columns of a wider buffer
    if op == "gram":
        # depth -1: the library chooses the Strassen levels; 1: the caller asks for one
        c["depth"] = 1 if dtype in ("f64", "f32") and rng.random() < 0.15 else -1
    if op in ("atb", "normal_solve", "project"):
        c["nrhs"] = rng.choice([1, 1, 2, 4, 9])
    return c


def _torch_dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _uniform(g, m, n, dtype, pad=0):
    buf = torch.rand((m, n + pad), generator=g, dtype=dtype, device="cuda")
    buf.mul_(2.0).sub_(1.0)
    return buf[:, :n]


def _pack(full):
    """Row-major packed lower triangle of a square matrix."""
    n = full.shape[0]
    i = torch.arange(n, device=full.device)
    return full[i[:, None] >= i[None, :]]


def _factor(g, n, dtype):
    """A factor as the Gram matrix of a 2 n x n matrix of N(0, 1) entries has
    it (Bartlett's decomposition): N(0, 1) below the diagonal, on it the
    lengths of vectors of 2 n - i such entries (their mean)."""
    full = torch.randn((n, n), generator=g, dtype=torch.float64, device="cuda").tril_(-1)
    full.diagonal().copy_(torch.sqrt(2.0 * n - torch.arange(n, device="cuda", dtype=torch.float64)))
    return full.to(dtype)


def _requests(case):
    """Shapes of the serving stream: m and n log-uniform."""
    r = random.Random(case["shapes"])
    return [(_log(r, 1024, 65536), _log(r, 64, 4096)) for _ in range(case["count"])]


def _inputs(case, seed):
    g, dt, op = _gen(seed), _torch_dtype(case), case["op"]
    if op in ("gram", "gram_rows"):
        return {"A": _uniform(g, case["m"], case["n"], dt, case["pad"])}
    if op == "cholesky":
        A = _uniform(g, 2 * case["n"], case["n"], dt)
        return {"C": _pack(A.t() @ A)}
    if op == "cholesky_solve":
        n = case["n"]
        B = torch.randn((n, case["nrhs"]), generator=g, dtype=dt, device="cuda") * math.sqrt(2.0 * n)
        return {"full": _factor(g, n, dt), "B": B}
    if op == "serve":
        return {"A": [torch.randn(s, generator=g, dtype=dt, device="cuda") for s in _requests(case)]}
    A = _uniform(g, case["m"], case["n"], dt)
    B = _uniform(g, case["m"], case["nrhs"], dt)
    return {"A": A, "B": B}


def prepare(case, seed):
    state = _inputs(case, seed)
    state["case"] = case
    if case["op"] == "cholesky":
        state["L"] = torch.empty_like(state["C"])
    if case["op"] == "cholesky_solve":
        state["L"] = _pack(state.pop("full"))
        state["X"] = torch.empty_like(state["B"])
    if case["op"] in ("cholesky", "normal_solve", "project"):
        state["info"] = torch.empty(1, dtype=torch.int32, device="cuda")
    if case["op"] == "serve":
        # room for the whole burst, as a server sized for its traffic has
        bytes_ = sum(4 * m * n + 4 * P.tri(n) for m, n in _requests(case))
        torch.cuda.synchronize()  # the server reads the inputs on its own streams
        state["server"] = serving.Server(2 * bytes_ + (1 << 30))
    return state


def run(state):
    c = state["case"]
    op = c["op"]
    if op == "gram":
        if c["depth"] < 0:
            return P.gram(state["A"], dtype=DTYPES[c["dtype"]])
        return P.gram(state["A"], dtype=DTYPES[c["dtype"]], max_depth=c["depth"])
    if op == "gram_rows":
        return P.gram_rows(state["A"], dtype=DTYPES[c["dtype"]])
    if op == "cholesky":
        state["L"].copy_(state["C"])
        return {"L": P.cholesky(state["L"], c["n"], info=state["info"]), "info": state["info"]}
    if op == "cholesky_solve":
        state["X"].copy_(state["B"])
        return P.cholesky_solve(state["L"], state["X"], c["n"])
    if op == "atb":
        return P.atb(state["A"], state["B"])
    if op == "normal_solve":
        return {"X": P.normal_solve(state["A"], state["B"], info=state["info"]), "info": state["info"]}
    if op == "project":
        return {"PB": P.project(state["A"], state["B"], info=state["info"]), "info": state["info"]}
    srv = state["server"]
    tickets = [srv.submit(a.shape[0], a.shape[1], P.F32, a=a) for a in state["A"]]
    return [srv.take(t, device=True) for t in tickets]


def work(case):
    op, es = case["op"], 8 if case["dtype"] == "f64" else 4
    if op == "serve":
        return {"bytes": float(sum(es * (m * n + P.tri(n)) for m, n in _requests(case))),
                "flops": float(sum(m * n * (n + 1) for m, n in _requests(case)))}
    if op in ("gram", "gram_rows"):
        m, n = (case["m"], case["n"]) if op == "gram" else (case["n"], case["m"])
        # the bfloat16 pairs are three products by definition
        return {"bytes": float(es * (m * n + P.tri(n))),
                "flops": float(m * n * (n + 1) * (3 if case["dtype"] == "bf16x3" else 1))}
    n = case["n"]
    if op == "cholesky":
        return {"bytes": float(2 * es * P.tri(n)), "flops": n ** 3 / 3.0}
    r = case["nrhs"]
    if op == "cholesky_solve":
        return {"bytes": float(es * (P.tri(n) + 2 * n * r)), "flops": 2.0 * n * n * r}
    m = case["m"]
    bytes_ = es * (m * n + m * r + (m if op == "project" else n) * r)
    flops = 2.0 * m * n * r
    if op != "atb":
        flops += m * n * (n + 1.0) + n ** 3 / 3.0 + 2.0 * n * n * r
    if op == "project":
        flops += 2.0 * m * n * r
    return {"bytes": float(bytes_), "flops": flops}


def _least_squares(A, B):
    A, B = A.double(), B.double()
    L = torch.linalg.cholesky((A.t() @ A).cpu())
    return torch.cholesky_solve((A.t() @ B).cpu(), L).to(A.device)


def exact(case, seed):
    x, op = _inputs(case, seed), case["op"]
    if op == "gram":
        A = x["A"].double()
        return _pack(A.t() @ A)
    if op == "gram_rows":
        A = x["A"].double()
        return _pack(A @ A.t())
    if op == "cholesky":
        full = torch.zeros((case["n"], case["n"]), dtype=torch.float64, device="cuda")
        i = torch.arange(case["n"], device="cuda")
        full[i[:, None] >= i[None, :]] = x["C"].double()
        return {"L": _pack(torch.linalg.cholesky(full.cpu())), "info": None}
    if op == "cholesky_solve":
        L = x["full"].double()
        Y = torch.linalg.solve_triangular(L, x["B"].double(), upper=False)
        return torch.linalg.solve_triangular(L.t(), Y, upper=True)
    if op == "atb":
        return x["A"].double().t() @ x["B"].double()
    if op == "normal_solve":
        return {"X": _least_squares(x["A"], x["B"]), "info": None}
    if op == "project":
        return {"PB": x["A"].double() @ _least_squares(x["A"], x["B"]), "info": None}
    return [_pack(a.double().t() @ a.double()) for a in x["A"]]
