"""Fine-level Galerkin product in work items: every (dimension, degree) instantiation, with blocks of one item, split
diagonal blocks and split off-diagonal blocks (which are also stored transposed), against the oracle's sparse
products.  Tolerance: the same products in another order, 1e-13 of the largest entry (the bar of the other Galerkin
tests)."""
import numpy as np
import pytest

import fixtures as F
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# (d, p', cells per axis, leaf size): boxes of about `leaf` points, so that a diagonal block lists about as many
# entries; pieces hold at least 64 of them
CASES = [(2, 0, 12, 16), (2, 0, 30, 300), (2, 1, 30, 64), (2, 1, 40, 900), (2, 2, 30, 200), (2, 3, 40, 300),
         (3, 0, 10, 100), (3, 1, 10, 500), (3, 2, 8, 2000), (3, 3, 10, 4000)]


@pytest.mark.parametrize("d,pc,N,leaf", CASES)
def test_galerkin_items(d, pc, N, leaf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    print(f"[gpu-case] galerkin items d={d} p'={pc} N={N} leaf={leaf}", flush=True)
    prob = F.structured_qp(d, N, 2 if d == 3 else 3, jitter=0.2 if d == 2 else 0.0, cfg=2)
    h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val,
                    P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_levels=2))
    ho = O.build_hierarchy(prob.coords, prob.scipy(), coarse_degree=pc, leaf_size=leaf, max_levels=2)
    import scipy.sparse as sp

    def check(scale):
        rp, cl, vl = h.export_level(1)
        got = sp.csr_matrix((vl, cl, rp))
        want = ho.levels[1].A.tocsr() * scale
        assert abs(got - want).max() <= 1e-13 * abs(want).max()
        assert abs(got - got.T).max() == 0.0 or abs(got - got.T).max() <= 1e-14 * abs(want).max()
    check(1.0)
    h.update_values(torch.from_numpy(prob.val * 0.5).to("cuda"))   # the partial blocks are rewritten
    check(0.5)
    h.close()
