"""Launches and copies of a batched solve: iteration budgets on both sides of a
captured graph's 32 iterations (the rest of a budget runs without the graph),
and nodes whose rows go in and out in several runs around infeasible ones."""
import pytest

from workloads import make_instance, make_nodes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("max_iter", [0, 1, 30, 31, 32, 63, 70])
def test_budget_does_not_depend_on_the_launches(dev, max_iter):
    """The same budget as one run of single launches and as graphs of 32 with a
    remainder: equal iteration counts, iterates and bounds up to the rounding of
    sums that a compacted product may order differently (1e-15 per sum, over at
    most 71 iterations far below 1e-9)."""
    import torch
    import paper_2603_01306_amd as pr
    inst = make_instance(n=512, p=256, corr=0.8, k_true=5, snr=5.0, loss=0, seed=12, storage="f32")
    ctx = pr.Context(torch.from_numpy(inst.Xcm).to(dev), torch.from_numpy(inst.y).to(dev), 0, max_batch=16)
    ctx.set_debug(pr.DEBUG_FORCE_BATCH)
    raw = make_nodes(inst.p, 9, seed=4, max_j0=20, max_j1=3)
    nodes = [pr.Node(5, 0.2, 2.0, J0=a, J1=b) for a, b in raw]
    for q in (0, 4, 8):   # infeasible: more fixed to one than k allows
        nodes[q] = pr.Node(1, 0.2, 2.0, J1=[3, 7])
    g = torch.Generator(device=dev).manual_seed(5)
    B0 = torch.zeros(9, inst.p, dtype=torch.float64, device=dev)
    for q in range(9):   # a start in the node's domain: off J0, inside the box
        free = [j for j in range(inst.p) if nodes[q].status(inst.p)[j] != 1][:5]
        B0[q, free] = 0.1 * torch.rand(5, generator=g, device=dev, dtype=torch.float64)
    kw = dict(rel_gap_tol=0.0, max_iter=max_iter, method=1)
    one, B1 = ctx.solve_batch(nodes, B0, check_every=4096, **kw)
    many, B2 = ctx.solve_batch(nodes, B0, check_every=32, **kw)
    for q in range(9):
        assert one[q]["status"] == many[q]["status"] == (pr.INFEASIBLE if q in (0, 4, 8) else pr.MAXITER)
        if q in (0, 4, 8):
            assert not bool(B1[q].any()) and not bool(B2[q].any())
            continue
        assert one[q]["iters"] == many[q]["iters"] == max_iter
        assert bool(B2[q].any())
        assert torch.linalg.norm(B1[q] - B2[q]) <= 1e-9 * torch.linalg.norm(B1[q])
        for key in ("lower_bound", "primal"):
            assert abs(one[q][key] - many[q][key]) <= 1e-9 * abs(one[q]["primal"])
    ctx.close()
