"""Timed cases of the library: what a program that uses it has it solve.

A case is a block-tridiagonal Hermitian positive definite problem (N blocks of
size m, k right-hand sides), an element type, and the call made on it:

* ``factor_solve``  factor and solve in one pass (plan and workspace kept);
* ``solve``         new right-hand sides against stored factors;
* ``adjoint``       factor and solve, then the gradients of A, B and y;
* ``refine``        FP32 levels, FP64 residuals and corrections to 1e-12;
* ``algorithm1``    the schedule that forms both half systems at each level.

``systems`` > 1 makes the case a ragged batch of independent systems.
"""
import math

import torch

from paper_1807_00370_amd import workloads
from paper_1807_00370_amd.solver import Solver

_DTYPE = {"c128": torch.complex128, "c64": torch.complex64, "r64": torch.float64,
          "r32": torch.float32}


def _case(name, call, dtype, N, m, k, graphs=False, matrix="random", systems=1):
    c = {"call": call, "dtype": dtype, "N": N, "m": m, "k": k, "graphs": graphs,
         "matrix": matrix, "systems": systems}
    return dict(c, name=name) if name else c


def listed():
    return [
        # one small solve inside a larger program: launches and latency count
        _case("tiny_c128", "factor_solve", "c128", 64, 4, 1),
        # a small problem solved again and again in the same buffers, replayed
        # from a recorded graph (time stepping)
        _case("small_graph_c128", "factor_solve", "c128", 4096, 16, 4, graphs=True),
        # many narrow blocks, one right-hand side (a banded system), odd count
        _case("narrow_c128", "factor_solve", "c128", 131071, 8, 1),
        # the large single system of the benchmark, in FP64 ...
        _case("large_c128", "factor_solve", "c128", 65536, 32, 16),
        # ... and as FP32 levels with FP64 refinement
        _case("large_refine", "refine", "c128", 65536, 32, 16),
        # new right-hand sides for a matrix factored before
        _case("resolve_c128", "solve", "c128", 16384, 32, 16),
        # the differentiable solve at the adjoint workload's size: one training step
        _case("adjoint_c128", "adjoint", "c128", 16384, 64, 32),
        # single precision, sizes that fit no tile: a training step
        _case("ragged_adjoint_c64", "adjoint", "c64", 9973, 23, 5),
        # large blocks of a size that fits no tile
        _case("wide_c128", "factor_solve", "c128", 1023, 200, 7),
        # the real 2D Poisson problem on a 256 x 4096 grid
        _case("poisson_r64", "factor_solve", "r64", 4096, 256, 1, matrix="poisson"),
        # independent systems of different shapes in one call
        _case("batch_c128", "factor_solve", "c128", 8192, 64, 16, systems=24),
        # the schedule without a back substitution per level
        _case("algorithm1_c128", "algorithm1", "c128", 2048, 32, 16),
    ]


def draw(rng):
    top = [work(c) for c in listed()]
    most = {q: max(w[q] for w in top) for q in ("bytes", "flops")}

    def log(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    while True:
        call = rng.choices(("factor_solve", "solve", "adjoint", "refine", "algorithm1"),
                           (5, 2, 2, 2, 1))[0]
        dtype = "c128"
        if call in ("factor_solve", "solve"):
            dtype = rng.choices(("c128", "c64", "r64", "r32"), (4, 2, 2, 1))[0]
        elif call == "adjoint":
            dtype = rng.choice(("c128", "c64"))
        N, m, k = log(32, 131072), log(2, 256), log(1, 64)
        matrix, systems, graphs = "random", 1, False
        if dtype == "r64" and rng.random() < 0.3:
            matrix = "poisson"
        if call == "algorithm1":
            N, m = log(32, 4096), log(2, 64)
        elif matrix == "random" and rng.random() < 0.2:
            systems, N, m, k = rng.randint(2, 24), log(256, 8192), log(8, 64), log(2, 16)
        if call == "factor_solve" and rng.random() < 0.3:
            graphs = True
        c = _case(None, call, dtype, N, m, k, graphs, matrix, systems)
        w = work(c)
        if w["bytes"] <= most["bytes"] and w["flops"] <= most["flops"]:
            return c


def _shapes(c):
    """(N, m, k) of each system; a batch spreads N, m and k below the case's."""
    if c["systems"] == 1:
        return [(c["N"], c["m"], c["k"])]
    ms = sorted({max(2, c["m"] // q) for q in (1, 2, 4, 8)})
    ks = sorted({1, max(1, c["k"] // 4), c["k"]})
    return workloads.batch_shapes(c["systems"], c["systems"] + c["N"],
                                  (max(1, c["N"] // 64), max(1, c["N"] // 2)), ms, ks)


def work(case):
    """Bytes and operations of the block Cholesky recurrence, the least known:
    every input read once (the lower triangle of A), every result written once."""
    real = case["dtype"] in ("r64", "r32")
    s = {"c128": 16, "c64": 8, "r64": 8, "r32": 4}[case["dtype"]]
    elems = mac = 0
    for N, m, k in _shapes(case):
        tri, mm, mk = m * (m + 1) // 2, m * m, m * k
        factor = m * mm / 6 + mm * m  # Cholesky; L \\ B and its product
        solve = 3 * mm * k            # two triangular solves, two block products
        matrix = N * tri + (N - 1) * mm
        if case["call"] == "solve":
            elems += matrix + 2 * N * mk
            mac += N * solve
        elif case["call"] == "adjoint":
            elems += matrix + (2 * N - 1) * mm + 4 * N * mk
            mac += N * (factor + 2 * solve + 3 * mm * k)
        else:
            elems += matrix + 2 * N * mk
            mac += N * (factor + solve)
    return {"bytes": s * elems, "flops": (2 if real else 8) * mac}


# ------------------------------------------------------------------- inputs


def _norms(B):
    """2-norms of the blocks by power iteration (a little below the true ones)."""
    v = torch.ones(B.shape[0], B.shape[2], 1, dtype=B.dtype, device=B.device)
    Bh = B.mH.contiguous()
    for _ in range(8):
        v = Bh @ (B @ v)
        v = v / torch.linalg.vector_norm(v, dim=1, keepdim=True)
    return torch.linalg.vector_norm(B @ v, dim=1).reshape(-1)


def _system(N, m, k, case, gen):
    """A, B, y in 64 bits: the block diagonally dominant Hermitian matrix of
    ``workloads.random_hpd`` (or its real case), or the 2D Poisson matrix."""
    real = case["dtype"] in ("r64", "r32")
    wide = torch.float64 if real else torch.complex128
    kw = {"dtype": wide, "device": "cuda", "generator": gen}
    y = torch.randn(N, m, k, **kw)
    if case["matrix"] == "poisson":
        one = torch.ones(m - 1, dtype=wide, device="cuda")
        A1 = 4 * torch.eye(m, dtype=wide, device="cuda") - torch.diag(one, 1) - torch.diag(one, -1)
        B1 = -torch.eye(m, dtype=wide, device="cuda")
        return A1.repeat(N, 1, 1), B1.repeat(N - 1, 1, 1), y
    B = torch.randn(N - 1, m, m, **kw) / math.sqrt(m)
    shift = torch.ones(N, dtype=torch.float64, device="cuda")
    if N > 1:
        nb = _norms(B)
        shift[1:] += nb
        shift[:-1] += nb
    A = torch.empty(N, m, m, dtype=wide, device="cuda")
    for a in range(0, N, 8192):
        e = min(N, a + 8192)
        M = torch.randn(e - a, m, m, **kw)
        A[a:e] = M @ M.mH.contiguous() / m
        del M
    A = (A + A.mH) / 2
    A.diagonal(dim1=1, dim2=2).add_(shift[:, None])
    return A.contiguous(), B, y


def _systems(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    for N, m, k in _shapes(case):
        A, B, y = _system(N, m, k, case, gen)
        gx = None
        if case["call"] == "adjoint":
            gx = torch.randn(N, m, k, dtype=y.dtype, device="cuda", generator=gen)
        yield A, B, y, gx


def _packed(case, seed):
    """The systems back to back in the case's type (one system keeps its shape)."""
    dt = _DTYPE[case["dtype"]]
    parts = [[t if t is None else t.to(dt) for t in q] for q in _systems(case, seed)]
    if len(parts) == 1:
        return parts[0]
    return [None if col[0] is None else torch.cat([t.reshape(-1) for t in col])
            for col in zip(*parts)]


def prepare(case, seed):
    A, B, y, gx = _packed(case, seed)
    Ns, ms, ks = zip(*_shapes(case))
    solver = Solver(Ns, ms, ks, dtype=_DTYPE[case["dtype"]],
                    precision="fp32_refine" if case["call"] == "refine" else "native",
                    schedule="pcr" if case["call"] == "algorithm1" else "cr")
    state = {"call": case["call"], "solver": solver, "A": A, "B": B, "y": y, "gx": gx, "x": None}
    if case["graphs"]:
        solver.set_graphs(True)  # a graph replays on the buffers it was recorded with
        state["x"] = torch.empty_like(y)
    if case["call"] == "solve":
        solver.factor(A, B)
    return state


def run(state):
    solver, A, B, y = state["solver"], state["A"], state["B"], state["y"]
    if state["call"] == "solve":
        return {"x": solver.solve(y), "info": solver.info}
    x = solver.factor_solve(A, B, y, state["x"])
    if state["call"] == "refine":
        return {"x": x}  # its info holds the measured residual
    if state["call"] == "adjoint":
        gA, gB, gy = solver.backward(x, state["gx"])
        return {"x": x, "info": solver.info, "gA": gA, "gB": gB, "gy": gy}
    return {"x": x, "info": solver.info}


# ------------------------------------------------------------- exact values


def _lower(L, G):
    """L \\ G in 64-row panels, each with the inverse of its diagonal tile."""
    m = L.shape[1]
    X = torch.empty_like(G)
    for a in range(0, m, 64):
        e = min(m, a + 64)
        r = G[:, a:e]
        if a:
            r = r - L[:, a:e, :a].contiguous() @ X[:, :a].contiguous()
        one = torch.eye(e - a, dtype=G.dtype, device=G.device).expand(L.shape[0], -1, -1)
        D = torch.linalg.solve_triangular(L[:, a:e, a:e].contiguous(), one.contiguous(),
                                          upper=False)
        X[:, a:e] = D @ r.contiguous()
    return X


def _upper(U, G):
    """U \\ G the same way: reversed rows and columns make it lower."""
    return _lower(U.flip(1, 2), G.flip(1)).flip(1)


def _eliminate(A, B, y):
    """x of the block-tridiagonal system by odd-even elimination, whole levels
    at a time on batched torch products."""
    n = A.shape[0]
    L = torch.linalg.cholesky(A[0::2].contiguous())
    g = _lower(L, y[0::2])
    nk, ne = n // 2, (n + 1) // 2
    x = torch.empty_like(y)
    if nk:
        P = _lower(L[:nk], B[0::2].mH.contiguous())
        Ph = P.mH.contiguous()
        A1 = A[1::2] - Ph @ P
        y1 = y[1::2] - Ph @ g[:nk]
        B1 = B[:0]
        if ne > 1:
            Q = _lower(L[1:], B[1::2].contiguous())
            Qh = Q.mH.contiguous()
            A1[:ne - 1] -= Qh @ Q
            y1[:ne - 1] -= Qh @ g[1:]
            if nk > 1:
                B1 = -(Ph[1:] @ Q[:nk - 1])
        x1 = _eliminate(A1, B1, y1)
        x[1::2] = x1
        g[:nk] -= P @ x1
        if ne > 1:
            g[1:] -= Q @ x1[:ne - 1]
    x[0::2] = _upper(L.mH.contiguous(), g)
    return x


def _times(A, B, x):
    r = A @ x
    if A.shape[0] > 1:
        r[1:] += B @ x[:-1]
        r[:-1] += B.mH.contiguous() @ x[1:]
    return r


def _solution(A, B, y):
    x = _eliminate(A, B, y)
    return x + _eliminate(A, B, y - _times(A, B, x))


def _sines(n):
    i = torch.arange(1, n + 1, dtype=torch.float64, device="cuda")
    S = torch.sin(torch.outer(i, i) * (math.pi / (n + 1))) * math.sqrt(2 / (n + 1))
    return S, 2 - 2 * torch.cos(i * (math.pi / (n + 1)))


def _poisson_solution(y):
    """The five-point Laplacian is diagonal in the sine basis of both axes."""
    N, m, k = y.shape
    Sm, lm = _sines(m)
    SN, lN = _sines(N)
    t = SN @ y.reshape(N, m * k)
    t = torch.einsum("ab,jbk->jak", Sm, t.reshape(N, m, k)) / (lN[:, None, None] + lm[:, None])
    t = torch.einsum("ab,jbk->jak", Sm, t)
    return (SN @ t.reshape(N, m * k)).reshape(N, m, k)


def exact(case, seed):
    out = {"x": [], "gA": [], "gB": [], "gy": []}
    narrow = case["dtype"] in ("c64", "r32")
    dt = _DTYPE[case["dtype"]]
    for A, B, y, gx in _systems(case, seed):
        if narrow:  # the values the call gets, in 64 bits
            wide = y.dtype
            A, B, y = A.to(dt).to(wide), B.to(dt).to(wide), y.to(dt).to(wide)
            gx = gx if gx is None else gx.to(dt).to(wide)
        if case["matrix"] == "poisson" and y.shape[0] <= 8192:  # dense sine transforms
            x = _poisson_solution(y)
        else:
            x = _solution(A, B, y)
        out["x"].append(x)
        if case["call"] == "adjoint":
            lam = _solution(A, B, gx)
            xh, lh = x.mH.contiguous(), lam.mH.contiguous()
            out["gA"].append((-(lam @ xh)).reshape(-1))
            out["gB"].append((-(lam[1:] @ xh[:-1] + x[1:] @ lh[:-1])).reshape(-1))
            out["gy"].append(lam)
    one = case["systems"] == 1
    got = {q: v[0] if one else torch.cat([t.reshape(-1) for t in v]) for q, v in out.items() if v}
    return got if case["call"] == "refine" else dict(got, info=None)
