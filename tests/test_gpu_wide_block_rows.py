"""Agglomerated levels with one very wide block row: a box coupled to every other one (512 boxes of 27 rows, 13,824 columns:
110 KB of float64 u, more than a workgroup's 64 KB of static LDS) keeps the block-row workgroup kernel, which holds u in
registers.  V-cycle against the oracle: 1e-11 in float64, 1e-5 in float32 (the bars of the other levels)."""
import numpy as np
import pytest
import scipy.sparse as sp

import fixtures as F
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def hub_problem():
    """3D Q1 31^3 (32^3 nodes, boxes of 4^3 of them) with a node of the central box coupled to one of each box."""
    prob = F.structured_qp(3, 31, 1)
    A = prob.scipy().tocsr()
    g = np.rint(prob.coords * 31).astype(int)
    one = np.flatnonzero(np.all(g % 4 == 1, axis=1))          # an interior node of each box
    assert len(one) == 512 and not prob.boundary[one].any()
    hub = one[np.argmin(np.abs(g[one] - 17).sum(1))]
    js = np.setdiff1d(one, A.indices[A.indptr[hub]:A.indptr[hub + 1]])
    v = np.full(len(js), 1e-3)
    C = sp.csr_matrix((np.concatenate([v, -v, -v, [v.sum()]]),
                       (np.concatenate([js, np.full(len(js), hub), js, [hub]]),
                        np.concatenate([js, js, np.full(len(js), hub), [hub]]))), shape=A.shape)
    A = (A + C).tocsr()
    A.sort_indices()
    return prob, A


@pytest.mark.parametrize("fp32", [0, 1])
def test_level_with_a_box_coupled_to_all_others(fp32):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    print(f"[gpu-case] wide block row fp32={fp32}", flush=True)
    prob, A = hub_problem()
    h = P.Hierarchy(prob.coords, A.indptr.astype(np.int64), A.indices.astype(np.int32), A.data,
                    P.Options(dim=3, coarse_degree=2, leaf_size=64, max_coarse_dofs=2000, vcycle_fp32=fp32))
    lv = h.info()
    assert [q["n"] for q in lv[1:]] == [13824, 1728]
    assert lv[1]["kernel"] == f"k_level_blockrow_wg<{'float' if fp32 else 'double'}>"
    print("us a launch", 1e3 * h.time_smoother_kernel(1, 200)[0], flush=True)
    ho = O.build_hierarchy(prob.coords, A, coarse_degree=2, leaf_size=64, max_coarse_dofs=2000)
    r = np.random.default_rng(1).standard_normal(prob.n)
    r[prob.boundary] = 0.0
    z = torch.zeros(prob.n, dtype=torch.float64, device="cuda")
    h.vcycle(torch.from_numpy(r).cuda(), z)
    want = O.vcycle(ho, r)
    assert np.linalg.norm(z.cpu().numpy() - want) <= (1e-5 if fp32 else 1e-11) * np.linalg.norm(want)
    h.close()
