"""Row counts of the batch's FP64 GEMM tiles (16 to 64 rows, one to three
tiles, and the padded ones): every node's iterate after a few batched steps
equals the single-node path's to summation order, for every storage type, both
losses and the Gram product."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROWS = [1, 16, 17, 32, 33, 48, 49, 64, 65, 80, 96, 97, 128, 129, 144, 145]


@pytest.mark.parametrize("dtype,loss,gram", [("float64", 0, False), ("float32", 0, False), ("bfloat16", 0, False),
                                             ("float32", 1, False), ("bfloat16", 1, False), ("float32", 0, True)])
def test_batched_rows_match_single_nodes(dev, dtype, loss, gram):
    import torch
    import paper_2603_01306_amd as pr
    n, p, k, its = 256, 384, 6, 4
    rng = np.random.default_rng(17)
    X = torch.from_numpy(rng.standard_normal((p, n))).to(dev).to(getattr(torch, dtype))
    u = X[:5].double().sum(0).cpu().numpy() + rng.standard_normal(n)
    y = torch.from_numpy(u if loss == 0 else np.where(u >= 0, 1.0, -1.0)).to(dev)
    ctx = pr.Context(X, y, loss, max_batch=max(ROWS))
    if gram:
        ctx.enable_gram()
    ctx.set_debug(pr.DEBUG_FORCE_BATCH)
    nodes = []
    for i in range(max(ROWS)):
        at = rng.permutation(p)
        nodes.append(pr.Node(k, 0.4 + 0.01 * i, 2.0, J0=at[: i % 11], J1=at[20: 20 + i % 4]))
    B0 = torch.from_numpy(0.01 * rng.standard_normal((len(nodes), p))).to(dev)
    for i, nd in enumerate(nodes):
        B0[i, torch.from_numpy(nd.J0.astype(np.int64)).to(dev)] = 0.0
    kw = dict(rel_gap_tol=0.0, max_iter=its)
    # the batch reports the last iterate: the single-node path's x^4 by a fifth step's start
    ref = {}
    for i in (0, 5, 15, 16, 31, 47, 63, 64, 79, 95, 127, 128, 143, 144):
        tr = torch.zeros(2 * (its + 1), dtype=torch.float64, device=dev)
        ctx.solve(nodes[i], beta0=B0[i], trace=tr, **kw)
        ref[i] = tr.cpu().numpy().reshape(-1, 2)[its]
    for m in ROWS:
        print(f"rows {m} {dtype} loss={loss} gram={gram}", flush=True)
        res, B = ctx.solve_batch(nodes[:m], B0=B0[:m], **kw)
        for i, (phi, psi) in ref.items():
            if i < m:
                assert res[i]["iters"] == its
                assert abs(res[i]["primal"] - phi) <= 1e-11 * abs(phi), (m, i)
                assert abs(res[i]["lower_bound"] - psi) <= 1e-11 * abs(phi), (m, i)
    ctx.close()
