"""The node step over several workgroups (p > 16384): per-iterate (Phi, Psi)
traces, the iterate and the counts against the FP64 oracle, on both sides of
the sizes where the entries per thread change, with ties in the dual's top
values, a top-kbar far wider than its window, no box, no free unit and a dense
warm start; and a repeated solve bit for bit."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

ITS = 12


def _instance(p, loss, seed, n=16):
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((p, n)).astype(np.float32)
    X[p // 3: p // 3 + 100] = X[p // 3]  # 100 equal columns: ties in the dual and in the prox
    X[-1] = X[0]
    u = X[:6].astype(np.float64).sum(axis=0) + 0.1 * rng.standard_normal(n)
    y = u if loss == 0 else np.where(u >= 0, 1.0, -1.0)
    return X, y, rng


@pytest.mark.parametrize("p,k,n0,n1,M,warm", [
    (16385, 8, 30, 2, 2.0, False),
    (16385, 900, 0, 0, float("inf"), True),   # 9 workgroups, the last with one entry
    (131072, 25, 64, 24, 2.0, False),         # 64 workgroups of 4 entries per thread
    (131073, 25, 64, 25, 2.0, True),          # 8 entries per thread; every unit fixed (kbar = 0)
    (262145, 10, 5, 0, float("inf"), False),  # 16 entries per thread
])
@pytest.mark.parametrize("loss", [0, 1])
def test_wide_node_traces(dev, p, k, n0, n1, M, warm, loss):
    import torch
    import paper_2603_01306_amd as pr
    print(f"wide node p={p} k={k} loss={loss}", flush=True)
    X, y, rng = _instance(p, loss, p + loss)
    ctx = pr.Context(torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev), loss)
    idx = rng.permutation(p)
    node = pr.Node(k, 0.7, M, J0=idx[:n0], J1=idx[n0:n0 + n1])
    st = node.status(p)
    X64 = X.astype(np.float64)
    L = (2.0 if loss == 0 else 0.25) * 1.01 * float(np.linalg.eigvalsh(X64.T @ X64).max())
    b0 = None
    if warm:
        b0 = 1e-4 * rng.standard_normal(p)
        b0[st == 1] = 0.0
    tr = torch.full((2 * (ITS + 1),), float("nan"), dtype=torch.float64, device=dev)
    kw = dict(rel_gap_tol=0.0, max_iter=ITS, L=L, want_zeta=True)
    start = None if b0 is None else torch.from_numpy(b0).to(dev)
    r = ctx.solve(node, beta0=start, trace=tr, **kw)
    ref = oracle.solve(X, y, loss, 0.7, M, k, status=st, L=L, tol=0.0, max_iter=ITS, trace_cap=ITS + 1, beta0=b0)
    assert (r["iters"], r["restarts"]) == (ITS, ref["restarts"])
    t = tr.cpu().numpy().reshape(-1, 2)
    ophi, opsi = ref["phi_trace"], ref["phi_trace"] - ref["trace"]
    fin = np.isfinite(ophi)
    assert np.array_equal(np.isfinite(t[:, 0]), fin)
    assert np.all(np.abs(t[fin, 0] - ophi[fin]) <= 1e-10 * np.abs(ophi[fin]))
    # an infinite primal value leaves no difference to take the oracle's bound from
    scale = np.abs(ophi[fin]).max() if fin.any() else np.abs(t[:, 1]).max()
    assert np.all(np.abs(t[fin, 1] - opsi[fin]) <= 1e-10 * scale)
    beta = r["beta"].cpu().numpy()
    if fin.any():
        assert np.abs(beta - ref["beta"]).max() <= 1e-10 * max(1.0, np.abs(ref["beta"]).max())
    psi = oracle.dual(X, y, r["zeta"].cpu().numpy(), loss, 0.7, M, k, status=st)
    assert abs(psi - r["lower_bound"]) <= 1e-11 * abs(psi)
    again = ctx.solve(node, beta0=start, **kw)
    assert (again["lower_bound"], again["primal"]) == (r["lower_bound"], r["primal"])
    assert torch.equal(again["beta"], r["beta"])
    ctx.close()
