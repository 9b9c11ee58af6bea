"""Chunk kernel of the fine level (rows padded to whole chunks of four entries, blocks of at most 768 chunks, 128 rows
and 511 distinct columns) at the edges of its blocks, forced through the tuning cache.

Every row-block kernel sums a row's products in the same order without fused multiply-adds, so the chunk kernel's
operator, V-cycles and solves equal CSR shape 0's bitwise; a row beyond the block limits is summed by the whole
workgroup instead, in another order, and is held to rounding (1e-14 for the operator, 1e-11 for the V-cycle, the bars
of the other shapes).
"""
import dataclasses

import numpy as np
import pytest

import fixtures as F

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CHUNK = 14


def _coupled(count):
    """2D Q1 30x30 plus a symmetric positive semi-definite coupling of one interior DoF with `count` - 9 others that
    are no neighbours of it: its row holds `count` entries."""
    import scipy.sparse as sp
    prob = F.structured_qp(2, 30, 1)
    A = prob.scipy().tocsr()
    free = np.flatnonzero(~prob.boundary)
    k = int(free[len(free) // 2])
    js = np.setdiff1d(free, A.indices[A.indptr[k]:A.indptr[k + 1]])[:count - 9]
    d = np.full(len(js), 1e-2)
    C = sp.csr_matrix((np.concatenate([d, d, d, [d.sum()]]),
                       (np.concatenate([np.full(len(js), k), js, js, [k]]),
                        np.concatenate([js, np.full(len(js), k), js, [k]]))), shape=A.shape)
    A = (A + C).tocsr()
    A.sort_indices()
    assert A.indptr[k + 1] - A.indptr[k] == count
    return prob.coords, A, 2


CASES = {
    "rows": lambda: _plain(2, 40, 1),        # 9 entries a row: the block's row limit
    "chunks": lambda: _plain(2, 24, 3),      # 16 to 49 entries: the chunk limit
    "columns": lambda: _plain(3, 8, 2),      # 27 to 125 entries: the column limit
    "one_block": lambda: _plain(2, 9, 1),    # 100 rows
    "row_510": lambda: _coupled(510),        # one row that nearly fills the column list ...
    "row_511": lambda: _coupled(511),        # ... that fills it
    "row_512": lambda: _coupled(512),        # ... and one beyond it, summed from memory
}


def _plain(d, N, p):
    prob = F.structured_qp(d, N, p, jitter=0.2 if d == 2 else 0.0, cfg=2)
    return prob.coords, prob.scipy().tocsr(), d


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_chunk_kernel(name, fp32, tmp_path, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    print(f"[gpu-case] chunk kernel {name} fp32={fp32}", flush=True)
    coords, A, d = CASES[name]()
    n = A.shape[0]
    base = P.Options(dim=d, coarse_degree=1, leaf_size=64, max_coarse_dofs=300, skip_leaf_level=int(d == 3),
                     vcycle_fp32=fp32)

    def handle(fine):
        return P.Hierarchy(coords, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                           dataclasses.replace(base, fine_kernel=fine))

    path = tmp_path / "tune.txt"
    monkeypatch.setenv("R3MG_TUNE_CACHE", str(path))
    handle(-1).close()
    key = [ln for ln in open(path) if "/fine1/" in ln][-1].rsplit(" ", 1)[0]
    with open(path, "a") as f:
        f.write(f"{key} {CHUNK + 100 * CHUNK}\n")
    h, ref = handle(-1), handle(0)
    assert h.info()[0]["kernel"].startswith("k_level_chunk<" + ("float" if fp32 else "double"))

    rng = np.random.default_rng(5)
    r = rng.standard_normal(n)
    bad = r.copy()
    bad[[n // 3, n // 2]] = np.inf, np.nan     # must reach exactly the rows that hold these columns
    b = A @ rng.standard_normal(n)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731

    def everything(q):
        out = []
        for v in (r, bad):
            y = torch.zeros(n, dtype=torch.float64, device="cuda")
            q.level_apply(0, t(v), y)
            out.append(y.cpu().numpy())
        z = torch.zeros(n, dtype=torch.float64, device="cuda")
        q.vcycle(t(r), z)
        x = torch.zeros(n, dtype=torch.float64, device="cuda")
        iters, _, ok = q.pcg(t(b), x, rtol=1e-10, maxit=300)
        assert ok
        return out + [z.cpu().numpy(), x.cpu().numpy()], int(iters[0])

    def compare(q, w):
        (a, ka), (c, kc) = everything(q), everything(w)
        assert np.linalg.norm(a[0] - A @ r) <= 1e-14 * np.linalg.norm(A @ r) or scaled
        assert np.array_equal(np.isfinite(a[1]), np.isfinite(c[1]))
        if name == "row_512":
            # another order in one row: rounding of the operator, float32 rounding through the float32 V-cycle
            for m, tol in ((0, 1e-14), (2, 1e-5 if fp32 else 1e-11), (3, 1e-9)):
                assert np.linalg.norm(a[m] - c[m]) <= tol * np.linalg.norm(c[m]), m
            assert abs(ka - kc) <= 1
        else:
            for m in range(4):
                assert np.array_equal(a[m], c[m], equal_nan=True), m
            assert ka == kc

    scaled = False
    compare(h, ref)
    # new values on the same pattern reach the chunked copies as well
    scaled = True
    vals = t(A.data * 1.75)
    h.update_values(vals)
    ref.update_values(vals)
    compare(h, ref)
    h.close()
    ref.close()
