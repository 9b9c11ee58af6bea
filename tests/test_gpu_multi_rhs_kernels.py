"""Multi-right-hand-side kernels forced through the tuning cache, against the lanes-per-row kernels (which the other tests
pin to the oracle): the box kernel of the agglomerated levels for every box size and column count, and the fine
level's chunk kernel in both block geometries, at the edges of its blocks.

Tolerances: the same products summed in another order.  The float64 V-cycle is held to 1e-11 and the float32 one to
1e-5 (the bars of the single-column V-cycles against the oracle and of float32 rounding through a V-cycle); solves to
1e-9 of each other.
"""
import dataclasses

import numpy as np
import pytest

import fixtures as F

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LANES, BOX, CHUNK = 8, 300, 400


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _vcycles(make, nrhs, path, monkeypatch, codes, n, seed=3, poison=False):
    """V-cycle outputs (nrhs, n) with each of the given {level: code} choices, read from the tuning cache."""
    monkeypatch.setenv("R3MG_TUNE_CACHE", str(path))
    r = np.random.default_rng(seed).standard_normal((nrhs, n))
    if poison:
        r[0, n // 3], r[nrhs - 1, n // 2] = np.inf, np.nan
    R = torch.from_numpy(r).to("cuda")
    h = make()
    h.vcycle(R, torch.empty_like(R))           # times every candidate once and writes the keys
    h.close()
    lines = [ln.rsplit(" ", 1)[0] for ln in open(path) if "/mr/" in ln]
    out = []
    for choice in codes:
        with open(path, "a") as f:
            for key in lines:
                level = int(key.split("/mr/")[1].split("/")[0])
                if level in choice:
                    f.write(f"{key} {choice[level]}\n")
        before = open(path).read()
        h = make()
        Z = torch.empty_like(R)
        h.vcycle(R, Z)
        Z2 = torch.empty_like(R)
        h.vcycle(R, Z2)
        torch.cuda.synchronize()
        assert open(path).read() == before      # the forced choices were valid: nothing was timed again
        assert torch.equal(Z.isnan(), Z2.isnan()) and torch.equal(torch.nan_to_num(Z), torch.nan_to_num(Z2))
        out.append(Z.cpu().numpy())
        h.close()
    return out


# (d, p', cells, leaf, largest coarsest level): boxes of 4, 9, 16, 8, 27 and 64 rows on at least one intermediate level
BOXES = [(2, 1, 30, 64, 300), (2, 2, 30, 64, 300), (2, 3, 30, 100, 300), (3, 1, 10, 150, 100), (3, 2, 10, 300, 300),
         (3, 3, 10, 700, 200)]


@pytest.mark.parametrize("nrhs", [2, 3, 8, 16])
@pytest.mark.parametrize("d,pc,N,leaf,mc", BOXES)
def test_box_kernel(d, pc, N, leaf, mc, nrhs, tmp_path, monkeypatch):
    _need_gpu()
    import paper_2607_28235_amd as P
    prob = F.structured_qp(d, N, 2 if d == 3 else 3, jitter=0.2 if d == 2 else 0.0, cfg=2)
    for fp32 in (0, 1):
        print(f"[gpu-case] box kernel d={d} p'={pc} nrhs={nrhs} fp32={fp32}", flush=True)
        o = P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=mc, vcycle_fp32=fp32)
        make = lambda: P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, o)  # noqa: E731
        h = make()
        levels = range(1, h.nlevels - 1)
        h.close()
        assert len(levels) >= 1
        same = {0: LANES, -1: LANES}
        a, b = _vcycles(make, nrhs, tmp_path / f"t{fp32}", monkeypatch,
                        [{**same, **{l: LANES for l in levels}}, {**same, **{l: BOX for l in levels}}], prob.n)
        for j in range(nrhs):
            assert np.linalg.norm(a[j] - b[j]) <= (1e-5 if fp32 else 1e-11) * np.linalg.norm(a[j]), (j, fp32)


def _matrix(name):
    import scipy.sparse as sp
    if name == "q1":                            # 9 entries a row: the block's row limit
        prob = F.structured_qp(2, 40, 1, jitter=0.2, cfg=2)
        return prob.coords, prob.scipy().tocsr(), 2
    if name == "q3":                            # the chunk limit
        prob = F.structured_qp(2, 20, 3, jitter=0.2, cfg=2)
        return prob.coords, prob.scipy().tocsr(), 2
    if name == "3d":                            # the column limit
        prob = F.structured_qp(3, 8, 2)
        return prob.coords, prob.scipy().tocsr(), 3
    # one row of `count` entries: within, at and beyond the column lists of 383 and 639
    count = int(name[3:])
    prob = F.structured_qp(2, 30, 1)
    A = prob.scipy().tocsr()
    free = np.flatnonzero(~prob.boundary)
    k = int(free[len(free) // 2])
    js = np.setdiff1d(free, A.indices[A.indptr[k]:A.indptr[k + 1]])[:count - 9]
    v = np.full(len(js), 1e-2)
    C = sp.csr_matrix((np.concatenate([v, v, v, [v.sum()]]),
                       (np.concatenate([np.full(len(js), k), js, js, [k]]),
                        np.concatenate([js, np.full(len(js), k), js, [k]]))), shape=A.shape)
    A = (A + C).tocsr()
    A.sort_indices()
    return prob.coords, A, 2


@pytest.mark.parametrize("nrhs", [2, 4, 5, 16])
@pytest.mark.parametrize("name", ["q1", "q3", "3d", "row383", "row384", "row639", "row640"])
def test_chunk_kernel(name, nrhs, tmp_path, monkeypatch):
    _need_gpu()
    import paper_2607_28235_amd as P
    coords, A, d = _matrix(name)
    n = A.shape[0]
    for fp32 in (0, 1):
        print(f"[gpu-case] chunk kernel {name} nrhs={nrhs} fp32={fp32}", flush=True)
        o = P.Options(dim=d, coarse_degree=1, leaf_size=64, max_coarse_dofs=300, skip_leaf_level=int(d == 3),
                      vcycle_fp32=fp32)
        make = lambda: P.Hierarchy(coords, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data, o)  # noqa: E731
        h = make()
        rest = {l: LANES for l in range(1, h.nlevels - 1)}
        h.close()
        for poison in (False, True):
            out = _vcycles(make, nrhs, tmp_path / f"t{fp32}{int(poison)}", monkeypatch,
                           [{**rest, 0: c, -1: c} for c in (LANES, CHUNK, CHUNK + 1)], n, poison=poison)
            for z in out[1:]:
                for j in range(nrhs):
                    if poison and j in (0, nrhs - 1):   # an infinity or NaN reaches the same entries of its column only
                        assert np.array_equal(np.isfinite(z[j]), np.isfinite(out[0][j]))
                        continue
                    assert np.linalg.norm(z[j] - out[0][j]) <= (1e-5 if fp32 else 1e-11) * np.linalg.norm(out[0][j])

    # the float64 operator of a block solve through the same kernel, new values included
    path = tmp_path / "solve"
    monkeypatch.setenv("R3MG_TUNE_CACHE", str(path))
    B = torch.from_numpy((A @ np.random.default_rng(1).standard_normal((n, nrhs))).T.copy()).to("cuda")
    h = make()
    h.vcycle(B, torch.empty_like(B))
    h.close()
    keys = [ln.rsplit(" ", 1)[0] for ln in open(path) if "/mr/0/" in ln or "/mr/-1/" in ln]
    sols = []
    for c in (LANES, CHUNK, CHUNK + 1):
        with open(path, "a") as f:
            for k in keys:
                f.write(f"{k} {c}\n")
        h = make()
        for vals in (A.data, 1.5 * A.data):
            if vals is not A.data:
                h.update_values(torch.from_numpy(vals).to("cuda"))
            X = torch.zeros_like(B)
            _, _, ok = h.pcg(B, X, rtol=1e-11, maxit=300)
            assert ok
            sols.append(X.cpu().numpy())
        h.close()
    for k in (2, 4):
        assert np.linalg.norm(sols[k] - sols[0]) <= 1e-9 * np.linalg.norm(sols[0])
        assert np.linalg.norm(sols[k + 1] - sols[1]) <= 1e-9 * np.linalg.norm(sols[1])
    assert np.linalg.norm(1.5 * sols[1] - sols[0]) <= 1e-8 * np.linalg.norm(sols[0])


# (d, p', cells, leaf): coarsest systems of 1, 4, 36, 216 and 1,728 unknowns, right above the leaves
@pytest.mark.parametrize("nrhs", [8, 11, 16])
@pytest.mark.parametrize("d,pc,N,leaf,nc", [(2, 0, 5, 300, 1), (2, 1, 5, 300, 4), (2, 2, 12, 200, 36),
                                            (3, 2, 8, 700, 216), (3, 2, 16, 700, 1728)])
def test_coarsest_solve_of_columns(d, pc, N, leaf, nc, nrhs):
    """Dense coarsest solve of several columns on the matrix cores, against one column at a time (another kernel)."""
    _need_gpu()
    import paper_2607_28235_amd as P
    prob = F.structured_qp(d, N, 2, jitter=0.0, cfg=2)
    R = np.random.default_rng(5).standard_normal((nrhs, prob.n))
    for fp32 in (0, 1):
        print(f"[gpu-case] coarsest nc={nc} nrhs={nrhs} fp32={fp32}", flush=True)
        o = P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=2000, vcycle_fp32=fp32)
        h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, o)
        assert h.nlevels == 2 and h.info()[1]["n"] == nc
        Z = torch.empty((nrhs, prob.n), dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(R).to("cuda"), Z)
        torch.cuda.synchronize()
        Z = Z.cpu().numpy()
        for c in range(nrhs):
            z = torch.empty(prob.n, dtype=torch.float64, device="cuda")
            h.vcycle(torch.from_numpy(R[c]).to("cuda"), z)
            torch.cuda.synchronize()
            z = z.cpu().numpy()
            assert np.linalg.norm(Z[c] - z) <= (1e-5 if fp32 else 1e-11) * np.linalg.norm(z)
        h.close()


# (d, p', cells, leaf): two-level float64 hierarchies on both sides of the size at which the packed inverse takes over
@pytest.mark.parametrize("d,pc,N,leaf,nc", [(2, 1, 8, 64, 32), (2, 1, 48, 40, 1024), (2, 2, 32, 64, 1152)])
def test_coarsest_solve_by_rows(d, pc, N, leaf, nc):
    """Two-level float64 V-cycle of one and of four columns against the oracle (the float64 V-cycle bar, 1e-11)."""
    _need_gpu()
    import oracle as O
    import paper_2607_28235_amd as P
    print(f"[gpu-case] coarsest by rows nc={nc}", flush=True)
    prob = F.structured_qp(d, N, 2, jitter=0.0, cfg=2)
    ho = O.build_hierarchy(prob.coords, prob.scipy(), coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=3000, max_levels=2)
    o = P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=3000, max_levels=2, vcycle_fp32=0)
    h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, o)
    assert h.nlevels == 2 and h.info()[1]["n"] == nc
    R = np.random.default_rng(6).standard_normal((4, prob.n))
    R[:, prob.boundary] = 0.0
    zo = np.stack([O.vcycle(ho, r) for r in R])
    for nr in (1, 4):
        Z = torch.empty((nr, prob.n), dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(R[:nr]).to("cuda"), Z)
        torch.cuda.synchronize()
        for c in range(nr):
            assert np.linalg.norm(Z[c].cpu().numpy() - zo[c]) <= 1e-11 * np.linalg.norm(zo[c])
    h.close()
