"""Performance cases of the library: what a program that uses it runs, from
the smallest solves to the full-size ones, through the public Python entry
points.

listed() names the cases followed over time, draw() makes one more case of
the same ranges, prepare() makes what a program holds before the call (device
matrices, plans, batches, a server with resident factors), run() is one pass,
work() the flops and bytes that pass cannot do without, exact() its result by
plain torch in binary64.

A case is a dict with "op" and that op's sizes:

  solve     L X = B ("lower"), L^T X = B ("transpose") or U X = B ("upper") on
            a kept plan; "kept" says whether the inverted diagonal blocks are
            kept too (many right-hand sides for one factor) or belong to the
            pass (a new factor each time)
  mixed     the 16-bit sweeps refined with exact residuals
  batch     uneven independent systems in one batched call, factors kept
  serve     a burst of requests on a server's resident factors
  chol, lu, lu_piv          the blocked factorizations, in place
  lu_solve, lu_piv_solve    A X = B in one call
"""
import math
import time

import torch

from paper_1612_01855_amd import trsm as T

DEV = "cuda"
FLAGS = {"lower": 0, "transpose": T.FLAG_TRANSPOSE, "upper": T.FLAG_UPPER}


def listed():
    return [
        # the smallest solve in use (the library's smoke size): launches and latency
        {"name": "solve_256x64_f64", "op": "solve", "n": 256, "k": 64, "precision": "f64",
         "problem": "lower", "kept": False},
        # a few columns against a kept factor, odd sizes, the transposed problem
        {"name": "solve_t_1000x7_f64", "op": "solve", "n": 1000, "k": 7, "precision": "f64",
         "problem": "transpose", "kept": True},
        # an ordinary ragged single-precision system given as an upper triangle
        {"name": "solve_u_3001x500_f32", "op": "solve", "n": 3001, "k": 500, "precision": "f32",
         "problem": "upper", "kept": False},
        # the tall factor with few right-hand sides: a chain of dependent steps
        {"name": "solve_16384x128_f64", "op": "solve", "n": 16384, "k": 128, "precision": "f64",
         "problem": "lower", "kept": False},
        # the full-size double-precision solve (the benchmark's own step)
        {"name": "solve_16384x16384_f64", "op": "solve", "n": 16384, "k": 16384,
         "precision": "f64", "problem": "lower", "kept": False},
        # half-precision sweeps refined to 1e-12
        {"name": "mixed_8192x8192_f16", "op": "mixed", "n": 8192, "k": 8192, "precision": "f16",
         "tolerance": 1e-12},
        # uneven single-precision systems in one batched call
        {"name": "batch_48_f32", "op": "batch", "count": 48, "nmax": 2048, "kmax": 512,
         "precision": "f32", "n0": 4096},
        # a burst of requests on a server with resident factors
        {"name": "serve_24_48", "op": "serve", "factors": 24, "requests": 48, "nmax": 4096,
         "kmax": 512, "precision": "f32", "kind": "triangular"},
        # the factorizations of the benchmark's suite
        {"name": "chol_4096", "op": "chol", "n": 4096},
        {"name": "lu_8192", "op": "lu", "n": 8192},
        {"name": "lu_piv_4096", "op": "lu_piv", "n": 4096},
        # A X = B for a general matrix in one call
        {"name": "lu_piv_solve_1000x10", "op": "lu_piv_solve", "n": 1000, "k": 10},
    ]


def _spread(rng, lo, hi):
    """An integer spread over the logarithm of [lo, hi]; two in three are
    taken as they fall (mostly odd), one in three on a multiple of 32."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    if rng.random() < 1 / 3 and v >= 64:
        v = v // 32 * 32
    return max(lo, min(hi, v))


def draw(rng):
    op = rng.choice(["solve", "solve", "solve", "mixed", "batch", "serve", "chol", "lu",
                     "lu_piv", "lu_piv_solve", "lu_solve"])
    if op == "solve":
        return {"op": op, "n": _spread(rng, 32, 16384), "k": _spread(rng, 1, 8192),
                "precision": rng.choice(["f64", "f64", "f32"]),
                "problem": rng.choice(["lower", "lower", "transpose", "upper"]),
                "kept": rng.random() < 0.5}
    if op == "mixed":
        return {"op": op, "n": _spread(rng, 1024, 8192), "k": _spread(rng, 64, 8192),
                "precision": rng.choice(["f16", "f16", "bf16"]),
                "tolerance": rng.choice([1e-12, 1e-12, 0.0])}
    if op == "batch":
        return {"op": op, "count": _spread(rng, 2, 64), "nmax": _spread(rng, 256, 2048),
                "kmax": _spread(rng, 16, 512), "precision": rng.choice(["f32", "f64"]),
                "n0": rng.choice([64, 512, 4096])}
    if op == "serve":
        return {"op": op, "factors": _spread(rng, 2, 24), "requests": _spread(rng, 1, 60),
                "nmax": _spread(rng, 512, 4096), "kmax": _spread(rng, 16, 512),
                "precision": rng.choice(["f32", "f32", "f64"]),
                "kind": rng.choice(["triangular", "triangular", "cholesky"])}
    if op in ("chol", "lu"):
        return {"op": op, "n": _spread(rng, 64, 10000)}
    if op == "lu_piv":
        return {"op": op, "n": _spread(rng, 64, 4096)}
    return {"op": op, "n": _spread(rng, 64, 3000), "k": _spread(rng, 1, 512)}


# ---- inputs -----------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, *shape):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float64)


def _lower(g, n):
    """A well-conditioned factor: diagonal U[1, 2], strict lower entries
    U[-1, 1] / n, zeros above."""
    L = torch.rand((n, n), generator=g, device=DEV, dtype=torch.float64)
    L.mul_(2.0 / n).sub_(1.0 / n).tril_(-1)
    L.diagonal().copy_(torch.rand(n, generator=g, device=DEV, dtype=torch.float64) + 1.0)
    return L


def _spd(g, n):
    G = _randn(g, n, 2 * n)
    A = G @ G.t().contiguous()
    A.mul_(1.0 / (2 * n))
    A.diagonal().add_(1.0)
    return A


def _dominant(g, n):
    """Strictly column diagonally dominant: elimination exchanges no row."""
    A = torch.rand((n, n), generator=g, device=DEV, dtype=torch.float64) * 2.0 - 1.0
    A.diagonal().zero_()
    A.diagonal().add_(A.abs().sum(dim=0) + 1.0)
    return A


def _shapes(case, count):
    """Sizes of a batch's systems or a server's factors and of the widths on
    them: log-uniform in [64, nmax] and [1, kmax], the same for every seed."""
    g = torch.Generator().manual_seed(count * 7919 + case["nmax"] * 31 + case["kmax"])
    u = torch.rand(count, 2, generator=g, dtype=torch.float64).tolist()
    return [(min(case["nmax"], int(round(64 * (case["nmax"] / 64) ** a))),
             min(case["kmax"], int(round(case["kmax"] ** b)))) for a, b in u]


def _requests(case):
    """(factor, width) of each request of a burst."""
    sizes = [n for n, _ in _shapes(case, case["factors"])]
    widths = [k for _, k in _shapes(case, case["requests"])]
    return sizes, [((5 * r + 3) % len(sizes), k) for r, k in enumerate(widths)]


def _inputs(case, seed):
    """The seeded matrices of a case, by name."""
    g, op = _gen(seed), case["op"]
    if op in ("solve", "mixed"):
        L, B = _lower(g, case["n"]), _randn(g, case["n"], case["k"])
        if case.get("problem") == "upper":
            L = L.t().contiguous()
        if case["precision"] == "f32":
            L, B = L.float(), B.float()
        return {"L": L, "B": B}
    if op == "batch":
        dt = torch.float32 if case["precision"] == "f32" else torch.float64
        return {"systems": [(_lower(g, n).to(dt), _randn(g, n, k).to(dt))
                            for n, k in _shapes(case, case["count"])]}
    if op == "serve":
        sizes, requests = _requests(case)
        factors = [_lower(g, n) for n in sizes]
        return {"factors": factors,
                "requests": [(f, _randn(g, sizes[f], k)) for f, k in requests]}
    n = case["n"]
    A = _spd(g, n) if op == "chol" else _dominant(g, n) if op in ("lu", "lu_solve") \
        else _randn(g, n, n)
    return {"A": A, "B": _randn(g, n, case["k"])} if "k" in case else {"A": A}


# ---- what a program keeps between calls --------------------------------------

class _Batch:
    """Systems with their kept inverted blocks, and the batch made of them."""

    def __init__(self, case, systems):
        self.systems, self.solvers, self.X = systems, [], []
        items = []
        for L, B in systems:
            n, k = B.shape
            s = T.Solver.create(n, k, case["precision"], case["n0"])
            s.invert(L)
            X = torch.empty_like(B)
            self.solvers.append(s)
            self.X.append(X)
            items.append(T.BatchItem(n, k, L.data_ptr(), n, s.linv_ptr, B.data_ptr(), k,
                                     X.data_ptr(), k))
        self.handle = T.trsm_batch_create(items, T.PRECISIONS[case["precision"]], case["n0"])
        self.workspace = torch.empty(T.trsm_batch_workspace_bytes(self.handle) + 256,
                                     dtype=torch.uint8, device=DEV)

    def run(self):
        T.trsm_batch_run(self.handle, (self.workspace.data_ptr() + 255) // 256 * 256,
                         torch.cuda.current_stream().cuda_stream, False)
        return self.X

    def __del__(self):
        if getattr(self, "handle", None):
            torch.cuda.synchronize()
            T.trsm_batch_destroy(self.handle)
            self.handle = None


class _Serving:
    """A server with its registered factors and a burst of requests."""

    def __init__(self, case, factors, requests):
        budget = (256 << 20) + sum(80 * B.numel() + (8 << 20) for _, B in requests)
        budget += sum(80 * (L.shape[0] + 64) ** 2 for L in factors)
        self.server = T.trsm_server_create(budget, 64)
        register = T.trsm_server_register_chol if case["kind"] == "cholesky" \
            else T.trsm_server_register_L
        torch.cuda.synchronize()
        ids = [register(self.server, L.data_ptr(), L.shape[0], L.shape[0], case["precision"])
               for L in factors]
        self.requests = [(ids[f], B, torch.empty_like(B)) for f, B in requests]

    def run(self):
        waiting = []
        for lid, B, X in self.requests:
            k = B.shape[1]
            waiting.append(T.trsm_serve_submit(self.server, lid, B.data_ptr(), k, k,
                                               X.data_ptr(), k))
        limit = time.monotonic() + 60.0
        while waiting:
            still = []
            for t in waiting:
                state, status, _ = T.trsm_serve_poll(self.server, t)
                if state == T.REQ_ERROR or (state == T.REQ_DONE and status != T.OK):
                    raise RuntimeError(f"request: {T.status_string(status)}")
                if state != T.REQ_DONE:
                    still.append(t)
            waiting = still
            if waiting:
                if time.monotonic() > limit:
                    raise RuntimeError("the server did not finish in time")
                time.sleep(5e-5)
        return [X for _, _, X in self.requests]

    def __del__(self):
        if getattr(self, "server", None):
            T.trsm_server_destroy(self.server)
            self.server = None


def prepare(case, seed):
    op, x = case["op"], _inputs(case, seed)
    state = {"case": case, "inputs": x}
    if op in ("solve", "mixed"):
        state["solver"] = T.Solver.create(case["n"], case["k"], case["precision"], 0,
                                          FLAGS[case.get("problem", "lower")],
                                          tolerance=case.get("tolerance", 0.0))
        if case.get("kept"):
            state["solver"].invert(x["L"])
    elif op == "batch":
        state["batch"] = _Batch(case, x["systems"])
    elif op == "serve":
        state["serving"] = _Serving(case, x["factors"], x["requests"])
    elif op in ("chol", "lu", "lu_piv"):
        make = {"chol": T.Cholesky, "lu": T.LU, "lu_piv": T.LUPiv}[op]
        state["factorization"] = make(case["n"])
        state["F"] = torch.empty_like(x["A"])
    return state


def run(state):
    case, x = state["case"], state["inputs"]
    op = case["op"]
    if op in ("solve", "mixed"):
        s = state["solver"]
        if not case.get("kept"):
            s.invert(x["L"])
        return s.solve(x["L"], x["B"])
    if op == "batch":
        return state["batch"].run()
    if op == "serve":
        return state["serving"].run()
    if op == "lu_solve":
        return T.lu_solve(x["A"], x["B"])
    if op == "lu_piv_solve":
        return T.lu_piv_solve(x["A"], x["B"])
    # the factorizations work in place: on a copy, as cholesky(A) and its
    # counterparts make one
    f, F = state["factorization"], state["F"]
    F.copy_(x["A"])
    f.factor(F)
    out = {"F": F, "Linv": f.linv_blocks()}
    if op == "lu":
        out["Uinv"] = f.uinv_blocks()
    if op == "lu_piv":
        out["ipiv"] = f.ipiv
    return out


# ---- what a pass cannot do without --------------------------------------------

def work(case):
    op = case["op"]

    def solves(shapes, size):
        return {"flops": float(sum(n * n * k for n, k in shapes)),
                "bytes": float(sum(size * (n * (n + 1) / 2 + 2 * n * k) for n, k in shapes))}

    if op in ("solve", "mixed"):
        return solves([(case["n"], case["k"])], 4 if case["precision"] == "f32" else 8)
    if op == "batch":
        return solves(_shapes(case, case["count"]), 4 if case["precision"] == "f32" else 8)
    if op == "serve":
        sizes, requests = _requests(case)
        w = solves([(sizes[f], k) for f, k in requests], 8)
        # each factor in use is read once, however many requests are on it
        w["bytes"] = 8.0 * (sum(sizes[f] * (sizes[f] + 1) / 2 for f in {f for f, _ in requests})
                            + sum(2 * sizes[f] * k for f, k in requests))
        w["flops"] *= 2 if case["kind"] == "cholesky" else 1
        return w
    n, k = case["n"], case.get("k", 0)
    if op == "chol":
        return {"flops": n ** 3 / 3, "bytes": 8.0 * n * (n + 1)}
    return {"flops": 2 * n ** 3 / 3 + 2.0 * n * n * k,
            "bytes": 8.0 * n * n * (1 if k else 2) + 16.0 * n * k}


# ---- the same by plain torch in binary64 ---------------------------------------

def _nb(case):
    """The documented default block size of a factorization."""
    n, op = case["n"], case["op"]
    if op == "lu_piv":
        nb, least = 256 if n <= 4096 else 512, 32
    else:
        nb, least = 512 if n >= 12288 else 256 if n >= 6144 else 128, 64
    return max(least, min(nb, 1 << (max(n, least) - 1).bit_length()))


def _block_inverses(F, nb, unit=False, upper=False):
    """Inverses of the nb x nb diagonal blocks of a triangle, a ragged last
    block padded with the identity."""
    n = F.shape[0]
    m = -(-n // nb)
    blocks = torch.eye(nb, dtype=F.dtype, device=F.device).repeat(m, 1, 1)
    for j in range(m):
        s = min(nb, n - j * nb)
        blocks[j, :s, :s] = F[j * nb:j * nb + s, j * nb:j * nb + s]
    eye = torch.eye(nb, dtype=F.dtype, device=F.device)
    return torch.stack([torch.linalg.solve_triangular(b, eye, upper=upper, unitriangular=unit)
                        for b in blocks])


def exact(case, seed):
    op, x = case["op"], _inputs(case, seed)

    def triangular(L, B, problem="lower"):
        L, B = L.double(), B.double()
        if problem == "transpose":
            L = L.t().contiguous()
        return torch.linalg.solve_triangular(L, B, upper=problem != "lower")

    if op in ("solve", "mixed"):
        return triangular(x["L"], x["B"], case.get("problem", "lower"))
    if op == "batch":
        return [triangular(L, B) for L, B in x["systems"]]
    if op == "serve":
        out = []
        for f, B in x["requests"]:
            X = triangular(x["factors"][f], B)
            if case["kind"] == "cholesky":
                X = triangular(x["factors"][f], X, "transpose")
            out.append(X)
        return out
    A = x["A"]
    n = A.shape[0]
    if op in ("lu_solve", "lu_piv_solve"):
        return torch.linalg.solve(A, x["B"])
    if op == "chol":
        L = torch.linalg.cholesky(A)
        return {"F": torch.tril(L) + torch.triu(A, 1), "Linv": _block_inverses(L, _nb(case))}
    nb = _nb(case)
    # on the host: LAPACK's exchanges are the ones meant (the device's own
    # factorization picks other rows); a column diagonally dominant matrix
    # keeps its rows under partial pivoting
    F = torch.linalg.lu_factor(A.cpu())[0].to(DEV)
    out = {"F": F, "Linv": _block_inverses(torch.tril(F, -1), nb, unit=True)}
    if op == "lu":
        out["Uinv"] = _block_inverses(torch.triu(F), nb, upper=True)
    else:
        out["ipiv"] = None
    return out
