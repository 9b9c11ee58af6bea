"""Group solves (r3mg_pcg_solve_group): every problem's outcome is that of its own solve.  A problem runs the same launches
on a stream of the library's instead of the caller's, so solutions, iteration counts and residuals are equal bit for
bit, whatever the others do: more problems than hardware queues, both V-cycle precisions in one group, a chunk that was
predicted too short or too long, a restart from the true residual, the iteration limit, eager launches, and inputs
that another stream is still writing."""
import dataclasses

import numpy as np
import pytest

import fixtures as F

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = [6, 8, 10, 7, 12, 9, 5]                              # cells per axis of 3D Q2 cubes: 1,331 to 15,625 DoFs


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _handles(kinds, **kw):
    """One handle per (cells, fp32) of kinds, with its own right-hand side."""
    import paper_2607_28235_amd as P
    hs, bs = [], []
    for k, (cells, fp32) in enumerate(kinds):
        prob = F.structured_qp(3, cells, 2)
        o = P.Options(dim=3, coarse_degree=1, leaf_size=150, max_coarse_dofs=300, vcycle_fp32=fp32, tune_cache=0)
        hs.append(P.Hierarchy(prob.coords, prob.row_ptr, prob.col, prob.val, dataclasses.replace(o, **kw)))
        b = np.random.default_rng(k).standard_normal(prob.n)
        b[prob.boundary] = 0.0
        bs.append(torch.from_numpy(b).cuda())
    return hs, bs


def _alone(hs, bs, **kw):
    """Each problem by itself: solutions, iterations, relative residuals, converged, restart-proof history."""
    out = []
    for h, b in zip(hs, bs):
        x = torch.zeros_like(b)
        it, rr, ok = h.pcg(b, x, **kw)
        out.append((x, int(it[0]), float(rr[0]), ok, h.history()))
    return out


def _group(hs, bs, **kw):
    import paper_2607_28235_amd as P
    xs = [torch.zeros_like(b) for b in bs]
    it, rr, ok = P.solve_group(hs, bs, xs, **kw)
    return xs, it, rr, ok


def _same(group, alone, hs):
    xs, it, rr, ok = group
    assert [int(k) for k in it] == [a[1] for a in alone]
    assert [float(r) for r in rr] == [a[2] for a in alone]
    assert ok == all(a[3] for a in alone)
    for x, a, h in zip(xs, alone, hs):
        assert torch.equal(x, a[0])
        assert np.array_equal(h.history(), a[4])


def _pairs(kinds, **kw):
    """Two sets of handles of the same problems, so that one set's predictions do not come from the other's solves."""
    hs, bs = _handles(kinds, **kw)
    return hs, _handles(kinds, **kw)[0], bs


@pytest.mark.parametrize("graph", [1, 0])
def test_mixed_precisions_and_more_problems_than_queues(graph):
    _need_gpu()
    print(f"[gpu-case] group of {len(N)} problems, both precisions, use_graph={graph}", flush=True)
    gs, hs, bs = _pairs([(n, k % 2) for k, n in enumerate(N)], use_graph=graph)
    # the first solve predicts three iterations, the second its own count, the others too few and too many
    for rtol in (1e-8, 1e-8, 1e-11, 1e-4, 1e-10):
        _same(_group(gs, bs, rtol=rtol, maxit=100), _alone(hs, bs, rtol=rtol, maxit=100), gs)


def test_one_member_at_the_iteration_limit():
    _need_gpu()
    print("[gpu-case] group: iteration limit", flush=True)
    gs, hs, bs = _pairs([(12, 1), (6, 0), (8, 1)])
    bs[1] = torch.zeros_like(bs[1])                          # converges at once
    for maxit in (0, 1, 3, 5):
        g, a = _group(gs, bs, rtol=1e-12, maxit=maxit), _alone(hs, bs, rtol=1e-12, maxit=maxit)
        assert not g[3] and not a[0][3] and a[1][3] and a[0][1] == maxit
        _same(g, a, gs)
    a = _alone(hs, bs, rtol=1e-6, maxit=100)
    most = max(q[1] for q in a)
    g, a = _group(gs, bs, rtol=1e-6, maxit=most - 1), _alone(hs, bs, rtol=1e-6, maxit=most - 1)
    assert not g[3] and sum(not q[3] for q in a) < len(a)    # some reach the limit, the others converge
    _same(g, a, gs)
    _same(_group(gs, bs, rtol=1e-10, maxit=100), _alone(hs, bs, rtol=1e-10, maxit=100), gs)


def test_member_that_restarts_from_its_true_residual():
    """At a tolerance below the rounding of the residual the recursion of the float32 members converges and their true
    residuals need not: one that does not restarts, which shows as a step of the residual history that falls by little or
    rises (every ordinary one is below 0.06 of the one before).  The float64 member beside them converges."""
    _need_gpu()
    print("[gpu-case] group: restart", flush=True)
    gs, hs, bs = _pairs([(10, 1), (8, 0), (12, 1), (7, 1)])
    x0 = [torch.randn(b.numel(), dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
          for b in bs]
    import paper_2607_28235_amd as P
    for rtol in (1e-13, 1e-15, 2e-16):
        alone = []
        for h, b, s in zip(hs, bs, x0):
            x = s.clone()
            it, rr, ok = h.pcg(b, x, rtol=rtol, maxit=60)
            alone.append((x, int(it[0]), float(rr[0]), ok, h.history()))
        xs = [s.clone() for s in x0]
        it, rr, ok = P.solve_group(gs, bs, xs, rtol=rtol, maxit=60)
        _same((xs, it, rr, ok), alone, gs)
    slow = [max(a[4][1:] / a[4][:-1]) > 0.1 for a in alone]
    assert any(slow[k] for k in (0, 2, 3)) and not slow[1] and alone[1][3]


def test_inputs_still_being_written_on_the_callers_stream():
    _need_gpu()
    print("[gpu-case] group: caller's stream", flush=True)
    gs, hs, bs = _pairs([(9, 1), (7, 0), (8, 1), (6, 1), (10, 0)])
    want = _alone(hs, bs, rtol=1e-10, maxit=100)
    import paper_2607_28235_amd as P
    side = torch.cuda.Stream()
    a = torch.randn(2048, 2048, device="cuda")
    for _ in range(3):
        late = [torch.full_like(b, float("nan")) for b in bs]
        xs = [torch.full_like(b, float("nan")) for b in bs]
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            c = a
            for _ in range(20):                              # some milliseconds before the vectors are written
                c = torch.tanh(c @ a)
            for q, b in zip(late, bs):
                q.copy_(b)
            for x in xs:
                x.zero_()
            it, rr, ok = P.solve_group(gs, late, xs, rtol=1e-10, maxit=100)
            twice = [2.0 * x for x in xs]                    # the caller's stream sees the solutions
        side.synchronize()
        _same((xs, it, rr, ok), want, gs)
        assert all(torch.equal(t, 2.0 * w[0]) for t, w in zip(twice, want))


def test_right_hand_side_that_is_another_problems_unknown():
    """b of one problem is x of another: every problem starts from the vectors as they were at the call."""
    _need_gpu()
    print("[gpu-case] group: shared vectors", flush=True)
    import paper_2607_28235_amd as P
    gs, hs, bs = _pairs([(9, 1), (9, 0), (9, 1)])
    first = [bs[1].clone(), bs[2].clone(), bs[0].clone()]    # the initial guesses
    want = []
    for h, b, s in zip(hs, (first[1], first[2], bs[2]), first):
        x = s.clone()
        it, rr, ok = h.pcg(b.clone(), x, rtol=1e-10, maxit=100)
        want.append((x, int(it[0]), float(rr[0]), ok, h.history()))
    xs = [s.clone() for s in first]
    it, rr, ok = P.solve_group(gs, [xs[1], xs[2], bs[2]], xs, rtol=1e-10, maxit=100)
    _same((xs, it, rr, ok), want, gs)
