"""Transfers of one right-hand side at every (dimension, p'): restriction and prolongation between the fine level and the
boxes (boxes of fewer and of more points than a workgroup's three waves, which take different prolongation kernels),
between agglomerated levels, and fused with the coarsest product, through the V-cycle against the oracle's.

Tolerances: the oracle's products in another order, 1e-11 in float64; float32 rounding through the V-cycle, 1e-5."""
import numpy as np
import pytest

import fixtures as F
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# (d, p', cells per axis, leaf size, largest coarsest level)
CASES = [(2, 0, 30, 16, 40), (2, 0, 40, 300, 10), (2, 1, 30, 64, 100), (2, 1, 40, 300, 60), (2, 2, 30, 64, 200),
         (2, 2, 40, 300, 150), (2, 3, 30, 100, 300), (2, 3, 40, 300, 200), (3, 0, 10, 30, 40), (3, 0, 10, 300, 4),
         (3, 1, 10, 150, 100), (3, 1, 10, 700, 20), (3, 2, 10, 300, 300), (3, 3, 10, 700, 200)]


@pytest.mark.parametrize("d,pc,N,leaf,mc", CASES)
def test_transfers(d, pc, N, leaf, mc):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    prob = F.structured_qp(d, N, 2 if d == 3 else 3, jitter=0.2 if d == 2 else 0.0, cfg=2)
    ho = O.build_hierarchy(prob.coords, prob.scipy(), coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=mc)
    r = np.random.default_rng(7).standard_normal(prob.n)
    r[ho.constrained] = 0.0
    want = O.vcycle(ho, r)
    for fp32, tol in ((0, 1e-11), (1, 1e-5)):
        print(f"[gpu-case] transfers d={d} p'={pc} N={N} leaf={leaf} fp32={fp32}", flush=True)
        h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val,
                        P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=mc, vcycle_fp32=fp32))
        assert h.nlevels >= 3
        z = torch.zeros(prob.n, dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(r).to("cuda"), z)
        got = z.cpu().numpy()
        h.close()
        assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)


@pytest.mark.parametrize("nrhs", [2, 5, 16])
@pytest.mark.parametrize("d,pc,N,leaf,mc", CASES[1::2])
def test_transfers_of_several_columns(d, pc, N, leaf, mc, nrhs):
    """The several-column transfers (matrix-core restriction, boxes split over workgroups), every column against the
    oracle's V-cycle of it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    prob = F.structured_qp(d, N, 2 if d == 3 else 3, jitter=0.2 if d == 2 else 0.0, cfg=2)
    ho = O.build_hierarchy(prob.coords, prob.scipy(), coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=mc)
    r = np.random.default_rng(8).standard_normal((nrhs, prob.n))
    r[:, ho.constrained] = 0.0
    want = [O.vcycle(ho, r[j]) for j in range(nrhs)]
    for fp32, tol in ((0, 1e-11), (1, 1e-5)):
        print(f"[gpu-case] transfers d={d} p'={pc} leaf={leaf} nrhs={nrhs} fp32={fp32}", flush=True)
        h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val,
                        P.Options(dim=d, coarse_degree=pc, leaf_size=leaf, max_coarse_dofs=mc, vcycle_fp32=fp32))
        R = torch.from_numpy(r).to("cuda")
        Z = torch.zeros_like(R)
        h.vcycle(R, Z)
        got = Z.cpu().numpy()
        h.close()
        for j in range(nrhs):
            assert np.linalg.norm(got[j] - want[j]) <= tol * np.linalg.norm(want[j]), j
