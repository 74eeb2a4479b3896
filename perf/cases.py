"""Workloads of the solver, each one pass through its public entry points.

`listed()` names the cases, `draw(rng)` gives more of the same ranges,
`prepare(case, seed)` makes on the GPU what a program has in hand before the
call, `run(state)` is one pass, `work(case)` what the pass cannot do without
and `exact(case, seed)` the results in 64 bits by plain torch.

Kinds of case:
  lu      lu_factor of a copy of A, then lu_solve: a dense system solved once
  solve   lu_solve alone on factors that the program keeps (many right-hand
          sides over time against one matrix)
  grad    the differentiable solve, forward and backward
  mxp     the mixed-precision solve (conversion, low-precision LU, FP64
          refinement), from a stored matrix or from a seed
  update  the trailing update C -= A B or the outer product C = -A B^T alone

Matrices: "uniform" entries in [-0.5, 0.5) (the benchmark recipe, up to
n = 1024); "shifted", the same with sqrt(n) / 2 added on the diagonal and the
rows permuted (larger systems: every column still needs its interchange, and
the solution is determined to the accuracy of the comparison); "dominant",
the recipe of the mixed-precision benchmark (diagonal = sum of the row's other
magnitudes), for the factorizations without pivoting.
"""

import math

import torch

from paper_2604_09517_amd import api, autograd

# -------------------------------------------------------------------- cases


def listed():
    return [
        # the smallest ordinary call: a system of a hundred unknowns, where
        # launches and waits are all that counts
        dict(name="lu_n100", kind="lu", n=100, nb=32, nrhs=1, trans=False),
        # the small benchmark configuration, N = 1024, NB = 64
        dict(name="lu_n1024", kind="lu", n=1024, nb=64, nrhs=1, trans=False),
        # a system of no convenient size, a few right-hand sides
        dict(name="lu_n5001_r3", kind="lu", n=5001, nb=256, nrhs=3, trans=False),
        # the headline benchmark, N = 32768, NB = 256
        dict(name="lu_n32768", kind="lu", n=32768, nb=256, nrhs=1, trans=False),
        # sixteen right-hand sides against kept factors
        dict(name="solve_n8192_r16", kind="solve", n=8192, nrhs=16, trans=False),
        # one transposed solve against kept factors, odd size (an adjoint)
        dict(name="solve_t_n2047_r1", kind="solve", n=2047, nrhs=1, trans=True),
        # the differentiable solve at its benchmark size, forward and backward
        dict(name="grad_fp64_n8192_r16", kind="grad", mode="fp64", n=8192, nb=256, nrhs=16),
        # its mixed-precision form as a layer of moderate size
        dict(name="grad_bf16_n1000_r2", kind="grad", mode="bf16_ir", n=1000, nb=128, nrhs=2),
        # the mixed-precision benchmark, BF16, N = 65536, NB = 512
        dict(name="mxp_bf16_n65536", kind="mxp", prec="bf16", n=65536, nb=512, nrhs=1,
             refine="gmres", pivot=False, seeded=False),
        # an odd size in FP16 with classical refinement, two right-hand sides
        dict(name="mxp_fp16_n3001_r2", kind="mxp", prec="fp16", n=3001, nb=256, nrhs=2,
             refine="classical", pivot=False, seeded=False),
        # the FP8 benchmark's recipe, regenerated from its seed, at the
        # largest size of which a pass stays near a second
        dict(name="mxp_fp8_seeded_n98304", kind="mxp", prec="fp8", n=98304, nb=1024, nrhs=1,
             refine="gmres", pivot=False, seeded=True),
        # the trailing update as a building block, ragged in every dimension
        dict(name="schur_6100x7003x300", kind="update", op="schur", m=6100, n=7003, k=300),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["lu", "lu", "solve", "solve", "grad", "mxp", "mxp", "update"])
    if kind == "lu":
        n = _log(rng, 64, 14000)
        return dict(kind="lu", n=n, nb=rng.choice([32, 64, 100, 128, 256]),
                    nrhs=rng.choice([1, 1, 2, 5, 16, 17]), trans=rng.random() < 0.25)
    if kind == "solve":
        return dict(kind="solve", n=_log(rng, 64, 14000),
                    nrhs=rng.choice([1, 1, 2, 3, 7, 16, 20]), trans=rng.random() < 0.5)
    if kind == "grad":
        if rng.random() < 0.5:
            return dict(kind="grad", mode="fp64", n=_log(rng, 64, 8192),
                        nb=rng.choice([64, 128, 256]), nrhs=rng.choice([1, 3, 16]))
        return dict(kind="grad", mode="bf16_ir", n=_log(rng, 64, 4000),
                    nb=rng.choice([64, 128, 256]), nrhs=rng.choice([1, 2, 4]))
    if kind == "mxp":
        prec = rng.choice(["bf16", "fp16", "fp8", "fp8_mx", "fp32"])
        pivot = prec in ("bf16", "fp32") and rng.random() < 0.25
        n = _log(rng, 256, 6000 if pivot or prec == "fp32" else 30000)
        nb = rng.choice([128, 256, 512]) if n < 16384 else rng.choice([512, 1024])
        return dict(kind="mxp", prec=prec, n=n, nb=nb, nrhs=rng.choice([1, 1, 2]),
                    refine=rng.choice(["gmres", "gmres", "classical"]), pivot=pivot,
                    seeded=not pivot and rng.random() < 0.4)
    return dict(kind="update", op=rng.choice(["schur", "outer"]), m=_log(rng, 64, 12000),
                n=_log(rng, 64, 12000), k=_log(rng, 16, 1024))


# ------------------------------------------------------------------- inputs


def _uniform(gen, *shape):
    return torch.rand(*shape, generator=gen, dtype=torch.float64, device="cuda").sub_(0.5)


def _matrix(gen, n, how):
    """Row j of the result is column j of the matrix (so its transpose view is
    the column-major matrix that the entry points take)."""
    cols = _uniform(gen, n, n)
    if how == "shifted":
        cols.diagonal().add_(0.5 * math.sqrt(n))
        cols = cols[:, torch.randperm(n, generator=gen, device="cuda")].contiguous()
    elif how == "dominant":
        cols.diagonal().zero_()
        cols.diagonal().copy_(torch.linalg.vector_norm(cols, ord=1, dim=0))
    return cols


def _vectors(gen, n, nrhs):
    """One right-hand side as a vector, several as a column-major matrix."""
    v = _uniform(gen, nrhs, n)
    return v[0] if nrhs == 1 else v.t()


def _i64(v):
    return v - (1 << 64) if v >= (1 << 63) else v


def _mix(z):
    """The SplitMix64 finaliser on int64 (wrapping products, logical shifts)."""
    z = z ^ ((z >> 30) & ((1 << 34) - 1))
    z = z * _i64(0xBF58476D1CE4E5B9)
    z = z ^ ((z >> 27) & ((1 << 37) - 1))
    z = z * _i64(0x94D049BB133111EB)
    return z ^ ((z >> 31) & ((1 << 33) - 1))


def _seeded_matrix(seed, n):
    """The dominant matrix of the seeded solve, from the generator's definition."""
    golden, mask = 0x9E3779B97F4A7C15, (1 << 64) - 1
    key = _mix(torch.tensor(_i64((seed + golden) & mask), device="cuda"))
    cols = torch.empty(n, n, dtype=torch.float64, device="cuda")
    step = max(1, (1 << 27) // n)
    for j in range(0, n, step):
        e = min(n, j + step)
        idx = torch.arange(j * n + 1, e * n + 1, device="cuda", dtype=torch.int64)
        h = (_mix(key + idx * _i64(golden)) >> 32) & 0xFFFFFFFF
        cols[j:e] = (h.to(torch.float64) * 2.0 ** -32 - 0.5).view(e - j, n)
    cols.diagonal().zero_()
    cols.diagonal().copy_(torch.linalg.vector_norm(cols, ord=1, dim=0))
    return cols


def _inputs(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    kind, n = case["kind"], case["n"]
    if kind == "update":
        m, k = case["m"], case["k"]
        B = _uniform(gen, n, k) if case["op"] == "schur" else _uniform(gen, k, n)
        return _uniform(gen, k, m).t(), B.t(), _uniform(gen, n, m).t()
    if kind == "mxp":
        b = _vectors(gen, n, case["nrhs"])
        if case["seeded"]:
            return None, b
        return _matrix(gen, n, "shifted" if case["pivot"] else "dominant").t(), b
    cols = _matrix(gen, n, "uniform" if n <= 1024 and kind != "grad" else "shifted")
    if kind == "grad":   # as torch programs hold them: row-major
        A = cols.t().contiguous()
        return A, _uniform(gen, n, case["nrhs"]), torch.randn(n, case["nrhs"], generator=gen,
                                                              dtype=torch.float64, device="cuda")
    return cols.t(), _vectors(gen, n, case["nrhs"])


def prepare(case, seed):
    s = {"case": case, "seed": int(seed)}
    kind, n = case["kind"], case["n"]
    if kind == "update":
        s["A"], s["B"], s["C0"] = _inputs(case, seed)
        s["C"] = api.fortran_empty(case["m"], n)
    elif kind == "grad":
        s["A"], s["B"], s["G"] = _inputs(case, seed)
        s["A"].requires_grad_(True)
        s["B"].requires_grad_(True)
    elif kind == "mxp":
        s["A"], s["B"] = _inputs(case, seed)
        s["X"] = torch.empty_like(s["B"])
        s["opts"] = api.mxp_options(prec=case["prec"], pivot=case["pivot"], nb=case["nb"],
                                    refine=case["refine"])
        s["work"] = torch.empty(api.mxp_workspace_bytes(n, s["opts"]), dtype=torch.uint8,
                                device="cuda")
        s["ipiv"] = torch.empty(n, dtype=torch.int32, device="cuda")
    else:
        s["A"], s["B"] = _inputs(case, seed)
        s["X"] = torch.empty_like(s["B"])
        s["ipiv"] = torch.empty(n, dtype=torch.int32, device="cuda")
        s["LU"] = api.fortran_empty(n, n)
        if kind == "solve":
            s["LU"].copy_(s.pop("A"))
            api.lu_factor(s["LU"], 256, s["ipiv"])
    return s


# --------------------------------------------------------------------- pass


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "update":
        if case["op"] == "schur":
            s["C"].copy_(s["C0"])
            return api.schur_update(s["C"], s["A"], s["B"])
        return api.outer_update(s["C"], s["A"], s["B"])
    if kind == "grad":
        X = autograd.solve(s["A"], s["B"], mode=case["mode"], nb=case["nb"])
        dA, dB = torch.autograd.grad(X, (s["A"], s["B"]), s["G"])
        return X.detach(), dA, dB
    if kind == "mxp":
        if case["seeded"]:
            api.mxp_solve_seeded(case["n"], s["seed"], 0, s["B"], X=s["X"], work=s["work"],
                                 opts=s["opts"])
        else:
            api.mxp_solve(s["A"], s["B"], X=s["X"], work=s["work"], ipiv=s["ipiv"],
                          opts=s["opts"])
        return s["X"], api.mxp_factors(s["work"], case["n"], case["prec"])
    s["X"].copy_(s["B"])
    if kind == "solve":
        return api.lu_solve(s["LU"], s["ipiv"], s["X"], trans=case["trans"])
    s["LU"].copy_(s["A"])
    api.lu_factor(s["LU"], case["nb"], s["ipiv"])
    api.lu_solve(s["LU"], s["ipiv"], s["X"], trans=case["trans"])
    return s["LU"], s["ipiv"], s["X"]


def work(case):
    kind, n = case["kind"], case["n"]
    if kind == "update":
        m, k = case["m"], case["k"]
        moved = m * k + k * n + (2 if case["op"] == "schur" else 1) * m * n
        return {"bytes": 8.0 * moved, "flops": 2.0 * m * n * k}
    r = case["nrhs"]
    if kind == "solve":
        return {"bytes": 8.0 * n * n + 16.0 * n * r + 4.0 * n, "flops": 2.0 * n * n * r}
    if kind == "grad":
        return {"bytes": 16.0 * n * n + 32.0 * n * r,
                "flops": 2.0 / 3.0 * n ** 3 + 6.0 * n * n * r}
    if kind == "mxp":
        stored = 4.0 if case["prec"] == "fp32" else 2.0
        return {"bytes": (stored + (0.0 if case["seeded"] else 8.0)) * n * n + 16.0 * n * r,
                "flops": 2.0 / 3.0 * n ** 3 + 4.0 * n * n * r}
    return {"bytes": 16.0 * n * n + 16.0 * n * r + 4.0 * n,
            "flops": 2.0 / 3.0 * n ** 3 + 2.0 * n * n * r}


# -------------------------------------------------------------------- exact


def _solve64(A, B, trans=False):
    M = A.t() if trans else A
    X = torch.linalg.solve(M.contiguous(), B.reshape(B.shape[0], -1))
    return X.reshape(B.shape)


def _jacobi64(A, B):
    """FP64 sweeps x += (b - A x) / diag: the dominant matrices contract by
    about 1 / sqrt(n) a sweep."""
    d = A.diagonal().clone()
    b = B.reshape(B.shape[0], -1)
    x = b / d[:, None]
    for _ in range(40):
        x += (b - A @ x) / d[:, None]
    return x.reshape(B.shape)


def exact(case, seed):
    kind, n = case["kind"], case["n"]
    if kind == "update":
        A, B, C = _inputs(case, seed)
        return C - A @ B if case["op"] == "schur" else -(A @ B.t())
    if kind == "grad":
        A, B, G = _inputs(case, seed)
        X, lam = _solve64(A, B), _solve64(A, G, True)
        return X, -(lam @ X.t()), lam
    A, B = _inputs(case, seed)
    if kind == "mxp":
        if case["pivot"]:
            return _solve64(A, B), None
        return _jacobi64(_seeded_matrix(int(seed), n).t() if A is None else A, B), None
    if kind == "solve":
        return _solve64(A, B, case["trans"])
    if n > 16384:
        return None
    # the factors by the host's LAPACK, where that takes seconds
    LU = torch.linalg.lu_factor(A.cpu().contiguous())[0] if n <= 8192 else None
    return LU, None, _solve64(A, B, case["trans"])
