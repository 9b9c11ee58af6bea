"""The 3D matrix-free cell kernel (one wave per Gauss slice of 64 cells) against the oracle's element loop, for every
degree, affine and multilinear cells, at cell counts below, at and past its tile of 64.

Tolerances: float64 to 1e-13 of the largest entry (the bar of the matrix-free operator against the oracle); the float32
V-cycle to 1e-5 of the float64 one (float32 rounding through a V-cycle).
"""
import numpy as np
import pytest

import fixtures as F
import oracle as O

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("jitter", [0.0, 0.15])
@pytest.mark.parametrize("N,p", [(2, 3), (3, 2), (4, 1), (4, 2), (4, 3), (5, 2), (9, 1)])
def test_cell_slices(N, p, jitter):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_28235_amd as P
    print(f"[gpu-case] matrix-free slices N={N} p={p} jitter={jitter}", flush=True)
    kappa = np.exp(np.random.default_rng(1).standard_normal(N ** 3))
    prob = F.structured_qp(3, N, p, jitter=jitter, cfg=6, kappa=kappa)
    x = np.random.default_rng(2).standard_normal(prob.n)
    yo = O.stiffness_apply(prob.coords, prob.cells, p, x, kappa=kappa, constrained=prob.boundary,
                           cdiag=np.ones(prob.n))
    r = np.random.default_rng(3).standard_normal(prob.n)
    r[prob.boundary] = 0.0
    z = []
    for fp32 in (0, 1):
        o = P.Options(dim=3, coarse_degree=1, leaf_size=200, max_coarse_dofs=300, vcycle_fp32=fp32)
        h = P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, o)
        h.set_matrix_free(prob.cells, p, kappa)
        y = torch.full((prob.n,), float("nan"), dtype=torch.float64, device="cuda")
        h.level_apply(0, torch.from_numpy(x).to("cuda"), y)
        zt = torch.zeros(prob.n, dtype=torch.float64, device="cuda")
        h.vcycle(torch.from_numpy(r).to("cuda"), zt)
        torch.cuda.synchronize()
        if not fp32:
            assert np.abs(y.cpu().numpy() - yo).max() <= 1e-13 * np.abs(yo).max()
        z.append(zt.cpu().numpy())
        h.close()
    assert np.linalg.norm(z[1] - z[0]) <= 1e-5 * np.linalg.norm(z[0])
