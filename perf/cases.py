"""The cases that this framework's speed is measured on.

A case is one pass through the public entry points as a user's program calls them: a PCG solve of an elliptic
problem on a handle the program keeps (one right-hand side, a block of them, a group of problems, the matrix-free
fine operator), a V-cycle handed to the program's own Krylov method, or a differentiable solve with its gradient.
The inputs are Q_p Lagrange discretisations of -div(kappa grad u) = f on [0,1]^d: structured or jittered cells,
Gauss-Lobatto nodes, Dirichlet rows as identity rows, assembled here with plain torch.  The seed decides the
vertices' jitter, the per-cell coefficient and the right-hand side, so another seed is another operator.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2607_28235_amd as P

DEV = "cuda" if torch.cuda.is_available() else "cpu"


# ------------------------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------------------------
def _case(kind, dim, cells, degree, coarse, leaf, **more):
    c = dict(kind=kind, dim=dim, cells=cells, degree=degree, coarse=coarse, leaf=leaf, skip_leaf=dim == 3, levels=0,
             coarsest=2000, steps=2, fp32=True, nrhs=1, rtol=1e-10, atol=0.0, jitter=False, kappa=False,
             by_cells=False, matrix_free=False)
    c.update(more)
    return c


def listed():
    return [
        # the smallest solve: the two-level problem of the smoke test, where launches and latency are everything
        _case("solve", 2, 16, 2, 1, 64, name="solve_2d_q2_16_f64", levels=2, steps=1, fp32=False),
        # the paper's experiments: a Q1 square, cell-based agglomeration, a 1e-6 reduction or 1e-9 absolute
        _case("solve", 2, 129, 1, 1, 8, name="solve_2d_q1_129_cells_f64", skip_leaf=True, fp32=False, rtol=1e-6,
              atol=1e-9, by_cells=True),
        # an ordinary 2D solve in float64 throughout, odd size
        _case("solve", 2, 101, 3, 2, 128, name="solve_2d_q3_101_f64", fp32=False, jitter=True),
        # the benchmark's own workload: 591,361 DoFs, float32 V-cycle in float64 CG
        _case("solve", 2, 256, 3, 2, 128, name="solve_2d_q3_256_f32", levels=4, jitter=True),
        # a large 3D solve with a coefficient (912,673 DoFs, 54 M nonzeros): the matrix fits no cache
        _case("solve", 3, 48, 2, 2, 256, name="solve_3d_q2_48_f32", kappa=True),
        # several right-hand sides at once: 16 columns on 3D Q3 (load cases, block methods)
        _case("solve", 3, 16, 3, 2, 256, name="batch16_3d_q3_16_f32", nrhs=16),
        # an odd number of columns in float64 on 2D Q2
        _case("solve", 2, 150, 2, 2, 128, name="batch5_2d_q2_150_f64", fp32=False, nrhs=5, jitter=True),
        # inversion / learning: assembly of A(kappa), numeric re-set-up, forward solve, adjoint solve, gradient
        _case("adjoint", 3, 24, 2, 2, 256, name="adjoint_3d_q2_24_f32", kappa=True),
        # several uneven problems solved together
        _case("group", 3, "13 16 21 25", 2, 2, 256, name="group4_3d_q2_f32"),
        # the fine level applied from the cells instead of the matrix
        _case("solve", 3, 40, 2, 2, 256, name="matrix_free_3d_q2_40_f32", matrix_free=True, kappa=True),
        # one V-cycle as the preconditioner of the caller's own Krylov loop
        _case("vcycle", 3, 29, 2, 2, 256, name="vcycle_3d_q2_29_f64", fp32=False),
    ]


# number of cells per axis by (dimension, degree): from a few hundred unknowns to about a quarter million
_RANGE = {(2, 1): (24, 480), (2, 2): (14, 240), (2, 3): (10, 160), (3, 1): (12, 56), (3, 2): (8, 30), (3, 3): (6, 16)}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "batch", "adjoint", "group", "matrix_free", "vcycle"])
    fp32 = rng.random() < 0.5
    dim = rng.choice([2, 3])
    degree = rng.choice([1, 2, 3])
    lo, hi = _RANGE[dim, degree]
    leaf = 128 if dim == 2 else 256
    coarse = rng.choice([1, 2])
    if kind == "adjoint":
        return _case("adjoint", 3, _log_int(rng, 8, 22), 2, coarse, 256, kappa=True, fp32=fp32)
    if kind == "group":
        sizes = [_log_int(rng, 8, 24) for _ in range(rng.randint(2, 4))]
        return _case("group", 3, " ".join(map(str, sizes)), 2, coarse, 256, fp32=fp32)
    if kind == "batch":
        return _case("solve", dim, _log_int(rng, lo, max(lo + 1, int(hi * 0.7))), degree, coarse, leaf, fp32=fp32,
                     nrhs=rng.randint(2, 16), jitter=dim == 2)
    n = _log_int(rng, lo, hi)
    if kind == "matrix_free":
        return _case("solve", dim, n, degree, coarse, leaf, fp32=fp32, matrix_free=True, kappa=True, jitter=dim == 2)
    if kind == "vcycle":
        return _case("vcycle", dim, n, degree, coarse, leaf, fp32=False, jitter=dim == 2, nrhs=rng.choice([1, 1, 3]))
    if dim == 2 and degree == 1 and rng.random() < 0.5:
        return _case("solve", 2, n, 1, 1, 8, skip_leaf=True, fp32=False, rtol=1e-6, atol=1e-9, by_cells=True)
    return _case("solve", dim, n, degree, coarse, leaf, fp32=fp32, jitter=dim == 2, kappa=dim == 3,
                 rtol=rng.choice([1e-10, 1e-8]))


# ------------------------------------------------------------------------------------------------------------
# Q_p discretisations of the unit square and cube
# ------------------------------------------------------------------------------------------------------------
def _nodes(p):
    s = 0.5 / math.sqrt(5.0)
    return {1: [0.0, 1.0], 2: [0.0, 0.5, 1.0], 3: [0.0, 0.5 - s, 0.5 + s, 1.0]}[p]


def _lagrange(nodes, s):
    """Values and derivatives (len(s), len(nodes)) of the Lagrange basis on `nodes` at the points s."""
    nodes, s = np.asarray(nodes), np.asarray(s)
    V = np.vander(nodes, increasing=True)
    C = np.linalg.inv(V)                                                 # column j: coefficients of basis j
    pw = np.vander(s, len(nodes), increasing=True)
    dp = np.concatenate([np.zeros((len(s), 1)), pw[:, :-1] * np.arange(1, len(nodes))], axis=1)
    return pw @ C, dp @ C


def _offsets(dim, p):
    """(local nodes, dim) grid offsets, x fastest."""
    k = p + 1
    a = np.arange(k ** dim)
    return np.stack([a // k ** m % k for m in range(dim)], axis=1)


@functools.lru_cache(maxsize=4)
def _grid(dim, N, p):
    """What the mesh's numbering alone decides: cells, corner vertices, boundary, and the CSR pattern."""
    M, W, offs = p * N + 1, 2 * p + 1, _offsets(dim, p)
    strides = M ** np.arange(dim)
    cg = np.stack([np.arange(N ** dim) // N ** m % N for m in range(dim)], axis=1)
    cells = torch.from_numpy(((cg[:, None, :] * p + offs) * strides).sum(-1)).to(DEV)
    verts = torch.from_numpy(((cg[:, None, :] + _offsets(dim, 1)) * (N + 1) ** np.arange(dim)).sum(-1)).to(DEV)
    n, nst = M ** dim, W ** dim
    g = torch.stack([torch.arange(n, device=DEV) // int(s) % M for s in strides], dim=1)
    boundary = ((g == 0) | (g == M - 1)).any(1)
    delta = torch.from_numpy((((offs[None] - offs[:, None]) + p) * W ** np.arange(dim)).sum(-1)).to(DEV)
    pat = torch.zeros(n * nst, dtype=torch.bool, device=DEV)
    for a in range(len(offs)):
        pat[cells[:, a, None] * nst + delta[a]] = True
    pat = pat.view(n, nst)
    dv = _offsets(dim, 2 * p) - p
    col = torch.arange(n, device=DEV)[:, None] + torch.from_numpy((dv * strides).sum(-1)).to(DEV)
    pat &= ~boundary[col.clamp(0, n - 1)]
    pat[boundary] = False
    pat[boundary, (nst - 1) // 2] = True
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = pat.sum(1).cumsum(0)
    return dict(cells=cells, verts=verts, boundary=boundary, delta=delta, pattern=pat,
                row_ptr=row_ptr, col=col[pat], row_ptr_host=row_ptr.cpu().numpy(),
                col_host=col[pat].to(torch.int32).cpu().numpy(), cells_host=cells.to(torch.int32).cpu().numpy())


def _element_matrices(X, dim, p):
    """Stiffness and mass matrices of multilinear cells with corners X (cells, 2^dim, dim), Gauss p+1."""
    gq, gw = np.polynomial.legendre.leggauss(p + 1)
    gq, gw = 0.5 * (gq + 1), 0.5 * gw
    offs, vo, q = _offsets(dim, p), _offsets(dim, 1), _offsets(dim, p)
    (V, D), (Vv, Dv) = _lagrange(_nodes(p), gq), _lagrange([0.0, 1.0], gq)
    w = np.prod(gw[q], axis=1)

    def tensor(A, B, o, m):
        return np.prod([(B if m == k else A)[q[:, k]][:, o[:, k]] for k in range(dim)], axis=0)

    val = torch.from_numpy(tensor(V, D, offs, -1)).to(DEV)
    grad = torch.from_numpy(np.stack([tensor(V, D, offs, m) for m in range(dim)], axis=-1)).to(DEV)
    vgrad = torch.from_numpy(np.stack([tensor(Vv, Dv, vo, m) for m in range(dim)], axis=-1)).to(DEV)
    K = torch.zeros(X.shape[0], len(offs), len(offs), dtype=torch.float64, device=DEV)
    Mm = torch.zeros_like(K)
    for i in range(len(q)):
        J = (X[:, :, :, None] * vgrad[i][None, :, None, :]).sum(1)          # dx_i / dxi_k
        det = torch.linalg.det(J)
        inv = torch.linalg.inv(J).contiguous()
        gphi = (grad[i][None, :, :, None] * inv[:, None]).sum(2)             # (cells, nodes, dim)
        wd = (det * w[i])[:, None, None]
        for m in range(dim):
            K += wd * gphi[:, :, m, None] * gphi[:, None, :, m]
        Mm += wd * val[i][None, :, None] * val[i][None, None, :]
    return 0.5 * (K + K.transpose(1, 2)), Mm


def _problem(case, N, seed, part=0):
    """Coordinates, CSR matrix (host and device values), right-hand sides and cell data of one problem."""
    dim, p = case["dim"], case["degree"]
    G = _grid(dim, N, p)
    rng = np.random.Generator(np.random.PCG64(np.random.SeedSequence((seed, N, part))))
    v = np.stack([np.arange((N + 1) ** dim) // (N + 1) ** m % (N + 1) for m in range(dim)], axis=1)
    x = v / N
    if case["jitter"]:
        inner = np.all((v > 0) & (v < N), axis=1)
        x[inner] += rng.uniform(-0.2 / N, 0.2 / N, size=(int(inner.sum()), dim))
    X = torch.from_numpy(x).to(DEV)[G["verts"]]
    K, Mm = _element_matrices(X if case["jitter"] else X[:1], dim, p)
    ncells = X.shape[0]
    kappa = torch.from_numpy(np.exp(rng.standard_normal(ncells) if case["kappa"] else np.zeros(ncells))).to(DEV)
    offs = _offsets(dim, p)
    ref = np.asarray(_nodes(p))[offs]
    vo = _offsets(dim, 1)
    shape = np.prod(np.where(vo[None] == 1, ref[:, None], 1 - ref[:, None]), axis=-1)
    coords = torch.empty(G["boundary"].numel(), dim, dtype=torch.float64, device=DEV)
    coords[G["cells"].reshape(-1)] = (torch.from_numpy(shape).to(DEV)[None, :, :, None] * X[:, None]).sum(2).reshape(-1, dim)
    prob = dict(n=coords.shape[0], G=G, Ke=K[0] if not case["jitter"] else K, kappa=kappa, val=_assemble(G, K, kappa),
                weights=torch.zeros(coords.shape[0], dtype=torch.float64, device=DEV))
    b = torch.zeros(case["nrhs"], prob["n"], dtype=torch.float64, device=DEV)
    for j in range(case["nrhs"]):                                            # b = M f, f ~ N(0, 1) at the nodes
        fe = torch.from_numpy(rng.standard_normal(prob["n"])).to(DEV)[G["cells"]]
        be = (Mm * fe[:, None, :]).sum(2)
        for a in range(len(offs)):
            b[j, G["cells"][:, a]] += be[:, a]
    we = Mm.sum(2)
    for a in range(len(offs)):
        prob["weights"][G["cells"][:, a]] += we[:, a]
    b[:, G["boundary"]] = 0.0
    prob["weights"][G["boundary"]] = 0.0
    prob["b"] = b if case["nrhs"] > 1 else b[0]
    prob["coords"] = coords.cpu().numpy()
    return prob


def _assemble(G, K, kappa):
    """CSR values of sum_e kappa_e K_e on the pattern, 1 on the Dirichlet rows."""
    pat = G["pattern"]
    S = torch.zeros(pat.numel(), dtype=torch.float64, device=DEV)
    for a in range(G["delta"].shape[0]):                                     # no two cells share their a-th node
        i = G["cells"][:, a, None] * pat.shape[1] + G["delta"][a]
        S[i] += K[:, a, :] * kappa[:, None]
    S = S.view(pat.shape)
    S[G["boundary"], (pat.shape[1] - 1) // 2] = 1.0
    return S[pat]


# ------------------------------------------------------------------------------------------------------------
# Preparation and passes
# ------------------------------------------------------------------------------------------------------------
def _options(case):
    return P.Options(dim=case["dim"], coarse_degree=case["coarse"], leaf_size=case["leaf"], max_levels=case["levels"],
                     max_coarse_dofs=case["coarsest"], skip_leaf_level=int(case["skip_leaf"]),
                     pre_steps=case["steps"], post_steps=case["steps"], vcycle_fp32=int(case["fp32"]))


def _sizes(case):
    return [int(s) for s in str(case["cells"]).split()]


def prepare(case, seed):
    probs = [_problem(case, N, seed, j) for j, N in enumerate(_sizes(case))]
    state = dict(case=case)
    if case["kind"] == "adjoint":
        q = probs[0]
        t = torch.from_numpy(q["coords"]).to(DEV)
        state["op"] = P.AdjointPoisson(q["coords"], q["G"]["row_ptr_host"], q["G"]["col_host"], q["val"].cpu().numpy(),
                                       q["G"]["cells_host"], q["Ke"].cpu().numpy(), q["weights"].cpu().numpy(),
                                       _options(case), rtol=case["rtol"], device=DEV)
        state["target"] = torch.sin(math.pi * t).prod(1)
        state["theta"] = q["kappa"].log()
        return state
    state["h"] = []
    for q in probs:
        h = P.Hierarchy(q["coords"], q["G"]["row_ptr_host"], q["G"]["col_host"], q["val"].cpu().numpy(), _options(case),
                        cells=q["G"]["cells_host"] if case["by_cells"] else None)
        if case["matrix_free"]:
            h.set_matrix_free(q["G"]["cells_host"], case["degree"], q["kappa"].cpu().numpy())
        state["h"].append(h)
    state["b"] = [q["b"] for q in probs]
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "adjoint":
        # one step of a gradient method on theta = log kappa: every pass forms a new kappa, as a step would
        theta = state["theta"].detach().requires_grad_()
        u = state["op"](theta.exp())
        loss = 0.5 * (u - state["target"]).square().sum()
        loss.backward()
        return {"u": u.detach(), "grad": theta.grad}
    if case["kind"] == "vcycle":
        z = torch.empty_like(state["b"][0])
        state["h"][0].vcycle(state["b"][0], z)
        return z
    xs = [torch.zeros_like(b) for b in state["b"]]
    if case["kind"] == "group":
        P.solve_group(state["h"], state["b"], xs, rtol=case["rtol"])
    else:
        state["h"][0].pcg(state["b"][0], xs[0], rtol=case["rtol"], atol=case["atol"])
    return xs


# ------------------------------------------------------------------------------------------------------------
# What a pass cannot do without, and its values in 64 bits
# ------------------------------------------------------------------------------------------------------------
def _size(dim, N, p):
    """(points, stored entries) of the matrix: interior points i couple with the interior points of their cells."""
    n, row = (p * N + 1) ** dim, 0
    for i in range(1, p * N):
        lo, hi = (i - p, i + p) if i % p == 0 else (i // p * p, i // p * p + p)
        row += min(hi, p * N - 1) - max(lo, 1) + 1
    return n, row ** dim + n - (p * N - 1) ** dim


def work(case):
    """Inputs read once (the matrix as CSR in float64, or the cells' connectivity and coefficient when the operator is
    matrix-free; the right-hand sides), outputs written once; the multiplications of the V-cycles' fine level (a
    Chebyshev step of degree 3 per smoothing step) and of CG, over nine iterations for a solve."""
    total = dict(bytes=0.0, flops=0.0)
    for N in _sizes(case):
        n, nnz = _size(case["dim"], N, case["degree"])
        k = case["nrhs"]
        matrix = N ** case["dim"] * (4 * (case["degree"] + 1) ** case["dim"] + 8) if case["matrix_free"] else 12 * nnz
        apply = 2.0 * nnz * k
        cycle = 6 * case["steps"] * apply
        if case["kind"] == "vcycle":
            b, f = matrix + 16 * n * k, cycle
        elif case["kind"] == "adjoint":
            b, f = matrix + 24 * n + 24 * N ** case["dim"], 2 * 9 * (cycle + apply)
        else:
            b, f = matrix + 16 * n * k, 9 * (cycle + apply)
        total["bytes"] += b
        total["flops"] += f
    return total


def _solver(G, val):
    """x = A^{-1} b by conjugate gradients with Jacobi scaling in float64, refined once from its true residual."""
    n = G["boundary"].numel()
    A = torch.sparse_csr_tensor(G["row_ptr"], G["col"], val, size=(n, n))
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), G["row_ptr"].diff())
    dinv = 1.0 / val[rows == G["col"]]

    def cg(b, tol):
        x, r = torch.zeros_like(b), b.clone()
        z = dinv * r
        p, rz, stop = z.clone(), r @ z, tol * float(b.norm())
        for k in range(20000):
            if k % 25 == 0 and float(r.norm()) <= stop:
                break
            q = A @ p
            a = rz / (p @ q)
            x += a * p
            r -= a * q
            z = dinv * r
            rz, old = r @ z, rz
            p = z + (rz / old) * p
        return x

    def solve(b):
        x = cg(b, 1e-13)
        return x + cg(b - A @ x, 1e-4)

    return solve


def exact(case, seed):
    if case["kind"] == "vcycle":
        return None      # B is defined by the library's own boxes, bounds and coarse operators
    probs = [_problem(case, N, seed, j) for j, N in enumerate(_sizes(case))]
    if case["kind"] == "adjoint":
        q = probs[0]
        solve = _solver(q["G"], q["val"])
        u = solve(q["weights"])
        lam = solve(u - torch.sin(math.pi * torch.from_numpy(q["coords"]).to(DEV)).prod(1))
        free = (~q["G"]["boundary"]).to(torch.float64)
        ue, le = (u * free)[q["G"]["cells"]], (lam * free)[q["G"]["cells"]]
        g = -((ue[:, None, :] * q["Ke"]).sum(2) * le).sum(1)
        return {"u": u, "grad": g * q["kappa"]}
    out = []
    for q in probs:
        solve = _solver(q["G"], q["val"])
        b = q["b"]
        out.append(solve(b) if b.dim() == 1 else torch.stack([solve(c) for c in b]))
    return out
