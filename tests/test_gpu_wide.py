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


@pytest.mark.parametrize("p", [1, 512, 513, 4096, 4097, 131072, 131073, 524288, 524289])
@pytest.mark.parametrize("ties", [False, True])
def test_prox_and_regularizer_at_shape_edges(dev, p, ties):
    """prox_{rho g_N}, g_N and g_N* where the number of workgroups and the
    entries per thread change (524289: the kernels over global memory), with
    many equal magnitudes and zeros and a cardinality past the gather's 64
    entries: 1e-12 of Algorithms 1 and 2, the tolerance of the other prox tests."""
    import torch
    import paper_2603_01306_amd as pr
    print(f"prox edges p={p} ties={ties}", flush=True)
    rng = np.random.default_rng(p + ties)
    v = rng.standard_normal(p)
    if ties:
        v = np.round(v, 1)  # about 80 magnitudes, exact zeros among them
    st = np.zeros(p, dtype=np.int8)
    if p > 100:
        idx = rng.permutation(p)
        st[idx[:20]] = oracle.ZERO
        st[idx[20:23]] = oracle.ONE
    k = min(300, max(4, p // 10))
    dv, ds = torch.from_numpy(v).to(dev), torch.from_numpy(st).to(dev)
    for rho, M in ((0.6, 2.0), (1.3, float("inf"))):
        x = pr.prox(dv, rho, k, M, ds).cpu().numpy()
        ref = oracle.prox_g(v, rho, k, M, st)
        assert np.abs(x - ref).max() <= 1e-12 * max(1.0, np.abs(ref).max())
        g, gs = pr.regularizer(torch.from_numpy(ref).to(dev), dv, k, M, ds)
        go, gso = oracle.g(ref, k, st), oracle.gstar(v, k, M, st)
        assert abs(g - go) <= 1e-12 * max(1.0, abs(go)) and abs(gs - gso) <= 1e-12 * max(1.0, abs(gso))
        assert pr.regularizer(None, dv, k, M, ds)[1] == gs
    bad = ds.clone()
    bad[p - 1] = 3
    out = torch.full_like(dv, 7.0)
    for fn in (lambda: pr.prox(dv, 0.5, k, 2.0, bad), lambda: pr.regularizer(dv, None, k, 2.0, bad),
               lambda: pr.prox_noalloc(dv, 0.5, k, 2.0, bad, out=out)):
        with pytest.raises(pr.PrError):
            fn()
    assert torch.all(out == 7.0)


def test_prox_from_many_threads_and_streams(dev):
    """More concurrent calls than the library keeps exchange areas for, each on
    a stream of its own: every result equals the serial one."""
    import threading
    import torch
    import paper_2603_01306_amd as pr
    gen = np.random.default_rng(3)
    cases = [torch.from_numpy(gen.standard_normal(20000 + 1000 * i)).to(dev) for i in range(12)]
    sts = [torch.zeros(v.numel(), dtype=torch.int8, device=dev) for v in cases]
    serial = [(pr.prox(v, 0.7, 12, 2.0, s), pr.regularizer(v, v, 12, 2.0, s)) for v, s in zip(cases, sts)]
    torch.cuda.synchronize()
    got = [None] * len(cases)

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                got[i] = (pr.prox(cases[i], 0.7, 12, 2.0, sts[i]), pr.regularizer(cases[i], cases[i], 12, 2.0, sts[i]))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for (x, g), (y, h) in zip(serial, got):
        assert torch.equal(x, y) and g == h


@pytest.mark.parametrize("p,k,n0,n1,M,warm", [
    (524288, 25, 64, 24, 2.0, False),          # the longest vector that workgroups share
    (524289, 25, 64, 24, 2.0, False),          # one workgroup over global memory
    (524289, 40, 0, 0, float("inf"), True),
])
@pytest.mark.parametrize("loss", [0, 1])
def test_node_traces_at_the_longest_shared_vector(dev, p, k, n0, n1, M, warm, loss):
    test_wide_node_traces(dev, p, k, n0, n1, M, warm, loss)


@pytest.mark.parametrize("p", [524288, 524289, 1048576])
@pytest.mark.parametrize("M", [2.0, float("inf")])
def test_noalloc_prox_at_the_longest_shared_vector(dev, p, M):
    """The prox without allocation over shared vectors and, past them, over its
    own scratch: pr_prox's output bit for bit."""
    import torch
    import paper_2603_01306_amd as pr
    print(f"noalloc prox p={p} M={M}", flush=True)
    rng = np.random.default_rng(p)
    v = np.round(rng.standard_normal(p), 3)
    st = np.zeros(p, dtype=np.int8)
    idx = rng.permutation(p)
    st[idx[:50]] = oracle.ZERO
    st[idx[50:57]] = oracle.ONE
    dv, ds = torch.from_numpy(v).to(dev), torch.from_numpy(st).to(dev)
    x = pr.prox(dv, 0.8, 300, M, ds)
    assert torch.equal(pr.prox_noalloc(dv, 0.8, 300, M, ds, out=torch.full_like(dv, float("nan"))), x)
    assert 250 < int((x != 0).sum()) < p and float(x[ds == oracle.ZERO].abs().max()) == 0.0
