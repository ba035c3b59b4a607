"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case is one call (or one short sequence of calls) of the public Python entry points, over the range of sizes that
this repository's own configurations, tests and benchmark use: the proximal operator and the regulariser at the
subroutine benchmark's smallest and largest shapes, root and child node relaxations of both losses from 500 x 200 to
32768 x 16384 and up to the 89989 columns of the widest design that the paper solves, batches of nodes, a whole branch
and bound, and the learned warm start's feature rows, forward pass and training step.

Designs follow workloads/synthetic.py's recipe (rows N(0, Sigma), Sigma_ij = corr^|i-j|, standardised columns, k unit
coefficients equally spaced, SNR 5), drawn on the GPU from the seed.
"""
import math

import torch

import paper_2603_01306_amd as pr

DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
VEC = {"f64": 2, "f32": 4, "bf16": 8}  # n is a multiple of this (16-byte loads of a column)
BYTES = {"f64": 8, "f32": 4, "bf16": 2}
LSQ, LOGISTIC = "least_squares", "logistic"


def _solve(name, n, p, dtype, loss, corr, k, lam, M, tol, method, evals, n0=0, n1=0, max_iter=2000):
    return dict(name=name, op="solve", n=n, p=p, dtype=dtype, loss=loss, corr=corr, k=k, lam=lam, M=M, tol=tol,
                method=method, evals=evals, n0=n0, n1=n1, max_iter=max_iter)


def _batch(name, m, n, p, dtype, loss, corr, k, lam, iters, gram=False):
    return dict(name=name, op="batch", m=m, n=n, p=p, dtype=dtype, loss=loss, corr=corr, k=k, lam=lam, M=2.0,
                iters=iters, gram=gram)


def listed():
    return [
        # the subroutine benchmark's smallest and largest vectors: prox of g_N, then g_N at its output and g_N*
        # (the smallest call a program makes: launches, copies and waits are all of it)
        dict(name="prox_p100", op="prox", p=100, k=10, M=1.0, rho=1.0, n0=0, n1=0),
        dict(name="prox_p102400", op="prox", p=102400, k=10, M=1.0, rho=1.0, n0=0, n1=0),
        # the small root relaxation, FP64 data, fixed step (the library's default method)
        _solve("root_ls_500x200_f64", 500, 200, "f64", LSQ, 0.5, 10, 1.0, 2.0, 1e-6, "fista", 140),
        # a branch-and-bound child of a mid-sized regression design with odd sizes (4459 rows padded to 4460, 4735
        # columns, M = 10), some coordinates already fixed, line search
        _solve("child_ls_4460x4735_f32", 4460, 4735, "f32", LSQ, 0.5, 10, 1.0, 10.0, 1e-6, "linesearch", 260, 40, 3),
        # the benchmark's root relaxation: least squares, line search, 1e-6 gap
        _solve("root_ls_16384x8192_f32", 16384, 8192, "f32", LSQ, 0.9, 20, 0.1, 2.0, 1e-6, "linesearch", 255),
        # the large logistic root, line search
        _solve("root_logistic_32768x16384_f32", 32768, 16384, "f32", LOGISTIC, 0.7, 15, 0.1, 2.0, 1e-6, "linesearch",
               77),
        # a few rows, very many columns (the widest design of the paper's tables): logistic node, k = 25, under an
        # iteration budget
        _solve("node_logistic_2300x89989_f32", 2300, 89989, "f32", LOGISTIC, 0.5, 25, 1.0, 2.0, 1e-4, "fista", 300, 200,
               5, 300),
        # 256 nodes of a tree together on the BF16 design, under an iteration budget
        _batch("batch256_ls_16384x8192_bf16", 256, 16384, 8192, "bf16", LSQ, 0.9, 20, 0.1, 48),
        # 48 logistic nodes together, FP32 data
        _batch("batch48_logistic_8192x4096_f32", 48, 8192, 4096, "f32", LOGISTIC, 0.7, 15, 0.1, 40),
        # a whole branch and bound, relaxations from the Gram matrix that the program formed once
        dict(name="bnb_gram_2048x2048_f32", op="bnb", n=2048, p=2048, dtype="f32", corr=0.5, k=10, lam=1.0, M=2.0),
        # feature rows of 32 children and the network's proposals for them (inference of the learned warm start)
        dict(name="features32_16384x8192_bf16", op="features", m=32, n=16384, p=8192, dtype="bf16", loss=LSQ, corr=0.9,
             k=20, lam=0.1, nnz=1200),
        # one training step of the network on about a million feature rows: gradient and Adam
        dict(name="train_step_rows1m", op="train", rows=1 << 20),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _fixed(rng, p, k):
    return rng.randrange(0, min(64, p // 4) + 1), rng.randrange(0, k)


def draw(rng):
    op = rng.choice(["prox", "solve", "solve", "solve", "batch", "features", "train"])
    if op == "prox":
        p, k = _log(rng, 100, 102400), rng.randrange(1, 26)
        n0, n1 = _fixed(rng, p, k)
        return dict(op="prox", p=p, k=k, M=rng.choice([1.0, 2.0, 10.0, math.inf]), rho=round(rng.uniform(0.01, 2.0), 4),
                    n0=n0, n1=n1)
    dtype = rng.choice(["f64", "f32", "f32", "bf16"])
    loss = rng.choice([LSQ, LOGISTIC])
    corr = rng.choice([0.1, 0.5, 0.7, 0.9])
    k = rng.choice([5, 10, 15, 20, 25])
    lam = rng.choice([0.1, 0.5, 1.0])
    if op == "solve":
        p = _log(rng, 200, 89989)
        n = max(500, min(_log(rng, 500, 32768), (1 << 27) // p)) // VEC[dtype] * VEC[dtype]
        n0, n1 = _fixed(rng, p, k)
        c = _solve("", n, p, dtype, loss, corr, k, lam, rng.choice([2.0, 10.0]), 1e-6,
                   "linesearch" if p <= 16384 and rng.random() < 0.5 else "fista", 120, n0, n1, 120)
        del c["name"]
        return c
    if op == "batch":
        n, p = 128 * _log(rng, 8, 96), 128 * _log(rng, 4, 48)
        gram = loss == LSQ and rng.random() < 0.3
        c = _batch("", rng.randrange(64, 129), n, p, dtype, loss, corr, k, lam, 32, gram)
        del c["name"]
        return c
    if op == "features":
        n, p = 128 * _log(rng, 8, 96), 128 * _log(rng, 4, 64)
        return dict(op="features", m=rng.randrange(4, 65), n=n, p=p, dtype=dtype, loss=loss, corr=corr, k=k, lam=lam,
                    nnz=rng.randrange(k, p // 4))
    return dict(op="train", rows=_log(rng, 10000, 1 << 20))


# ---------------------------------------------------------------- inputs


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _design(c, seed):
    """X as a (p, n) tensor (row j = column j of X) in the storage type, and y."""
    n, p, corr = c["n"], c["p"], c["corr"]
    g = _gen(seed, 1)
    work = torch.float64 if c["dtype"] == "f64" else torch.float32
    # blocks of B columns run the recursion side by side, then each block takes the share of its predecessor's last
    # column (corr^B is below FP32 rounding)
    B = max(1, math.ceil(-17.0 / math.log(corr)))
    nb = -(-p // B)
    X = torch.randn(nb, B, n, generator=g, device="cuda", dtype=work)
    s = math.sqrt(1.0 - corr * corr)
    X[1:, 0].mul_(s)
    for j in range(1, B):
        X[:, j].mul_(s).add_(X[:, j - 1], alpha=corr)
    last = X[:-1, B - 1].clone()
    for j in range(B):
        X[1:, j].add_(last, alpha=corr ** (j + 1))
    X = X.view(nb * B, n)[:p]
    X.sub_(X.mean(1, keepdim=True))
    X.div_(X.square().mean(1, keepdim=True).sqrt_())
    X = X.to(DTYPES[c["dtype"]]).contiguous() if c["dtype"] == "bf16" or nb * B != p else X
    support = torch.arange(c["k"], device="cuda") * (p // c["k"])
    signal = X[support].double().sum(0)
    noise = torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    noisy = signal + noise * (signal.var(unbiased=False) / 5.0).sqrt()
    y = noisy if c.get("loss", LSQ) == LSQ else torch.where(noisy >= 0, 1.0, -1.0).double()
    return X, y.contiguous()


def _index_sets(seed, salt, p, n0, n1):
    g = torch.Generator()
    g.manual_seed(1000003 * int(seed) + salt)
    idx = torch.randperm(p, generator=g)[: n0 + n1].numpy()
    return idx[:n0], idx[n0:]


def _nodes(c, seed):
    """Uneven nodes of a tree: |J0| in 0..64, |J1| in 0..k-1."""
    g = torch.Generator()
    g.manual_seed(1000003 * int(seed) + 7)
    nodes = []
    for q in range(c["m"]):
        n0 = int(torch.randint(0, 65, (1,), generator=g))
        n1 = int(torch.randint(0, c["k"], (1,), generator=g))
        J0, J1 = _index_sets(seed, 100 + q, c["p"], n0, n1)
        nodes.append(pr.Node(c["k"], c["lam"], c.get("M", 2.0), J0=J0, J1=J1))
    return nodes


def _vector_inputs(c, seed):
    g = _gen(seed, 3)
    v = torch.randn(c["p"], generator=g, device="cuda", dtype=torch.float64)
    w = torch.randn(c["p"], generator=g, device="cuda", dtype=torch.float64)
    st = torch.zeros(c["p"], dtype=torch.int8)
    J0, J1 = _index_sets(seed, 5, c["p"], c["n0"], c["n1"])
    st[torch.from_numpy(J0)] = pr.ZERO
    st[torch.from_numpy(J1)] = pr.ONE
    return v, w, st.cuda()


def _network(seed):
    """Parameters of a network in training and its Adam moments."""
    g = _gen(seed, 11)

    def u(*shape, bound):
        return (2.0 * torch.rand(*shape, generator=g, device="cuda") - 1.0) * bound

    P = torch.cat([u(512, bound=math.sqrt(6 / 8)), u(64, bound=0.1), u(4096, bound=math.sqrt(6 / 64)),
                   u(64, bound=0.1), u(64, bound=0.1 * math.sqrt(6 / 64)), u(1, bound=0.1)]).contiguous()
    m1 = 1e-3 * torch.randn(pr.MLP_NPARAM, generator=g, device="cuda")
    m2 = 1e-6 * (0.5 + torch.rand(pr.MLP_NPARAM, generator=g, device="cuda"))
    return P, m1, m2


def _parents(c, seed):
    """Sparse parent solutions and their children's, as nodes of a tree have them."""
    g = _gen(seed, 13)
    m, p = c["m"], c["p"]
    keep = torch.rand(m, p, generator=g, device="cuda") < c["nnz"] / p
    Bp = torch.where(keep, 0.05 * torch.randn(m, p, generator=g, device="cuda", dtype=torch.float64), 0.0)
    Bc = torch.where(keep, Bp + 0.005 * torch.randn(m, p, generator=g, device="cuda", dtype=torch.float64), 0.0)
    return Bp.contiguous(), Bc.contiguous()


def _train_rows(c, seed):
    g = _gen(seed, 17)
    F = torch.randn(c["rows"], pr.MLP_NFEAT, generator=g, device="cuda").to(torch.bfloat16)
    T = 0.1 * torch.randn(c["rows"], generator=g, device="cuda")
    return F, T


def _loss(c):
    return pr.LSQ if c.get("loss", LSQ) == LSQ else pr.LOGISTIC


def prepare(case, seed):
    c, op = case, case["op"]
    if op == "prox":
        v, w, st = _vector_inputs(c, seed)
        return dict(c=c, v=v, w=w, st=st)
    if op == "train":
        F, T = _train_rows(c, seed)
        P, m1, m2 = _network(seed)
        grad = torch.empty(pr.MLP_NPARAM + 1, device="cuda")
        work = torch.empty(pr.mlp_workspace(c["rows"]), device="cuda")
        return dict(c=c, F=F, T=T, P=P, m1=m1, m2=m2, grad=grad, work=work, step=100)
    X, y = _design(c, seed)
    ctx = pr.Context(X, y, _loss(c), max_batch=c.get("m", 1))
    if op == "solve":
        J0, J1 = _index_sets(seed, 5, c["p"], c["n0"], c["n1"])
        return dict(c=c, ctx=ctx, node=pr.Node(c["k"], c["lam"], c["M"], J0=J0, J1=J1))
    if op == "bnb":
        ctx.enable_gram()
        return dict(c=c, ctx=ctx, node=pr.Node(c["k"], c["lam"], c["M"]))
    if op == "batch":
        if c["gram"]:
            ctx.enable_gram()
        return dict(c=c, ctx=ctx, nodes=_nodes(c, seed))
    Bp, Bc = _parents(c, seed)
    return dict(c=c, ctx=ctx, nodes=_nodes(c, seed), Bp=Bp, Bc=Bc, P=_network(seed)[0])


METHOD = {"fista": pr.FISTA_GAP, "linesearch": pr.FISTA_BT_GAP}


def run(state):
    c, op = state["c"], state["c"]["op"]
    if op == "prox":
        x = pr.prox(state["v"], c["rho"], c["k"], c["M"], state["st"])
        g, gs = pr.regularizer(x, state["w"], c["k"], c["M"], state["st"])
        return {"x": x, "g": g, "gstar": gs}
    if op == "train":
        state["step"] += 1
        grad = pr.mlp_grad(state["P"], state["F"], state["T"], state["work"], state["grad"])
        pr.mlp_adam(state["P"], grad, state["m1"], state["m2"], state["step"])
        return {"grad": grad, "params": state["P"], "m1": state["m1"], "m2": state["m2"]}
    ctx = state["ctx"]
    if op == "solve":
        r = ctx.solve(state["node"], want_zeta=True, rel_gap_tol=c["tol"], method=METHOD[c["method"]],
                      max_iter=c["max_iter"])
        return {k: r[k] for k in ("lower_bound", "primal", "L", "iters", "trials", "restarts", "status", "beta",
                                  "zeta")}
    if op == "bnb":
        r, beta = ctx.bnb(state["node"], node_opts=dict(method=pr.FISTA_BT_GAP))
        return {k: r[k] for k in ("lower_bound", "upper_bound", "nodes_solved", "nodes_pruned", "status")} | {"beta": beta}
    if op == "batch":
        res, B = ctx.solve_batch(state["nodes"], rel_gap_tol=1e-6, method=pr.FISTA_BT_GAP, max_iter=c["iters"])
        out = {k: torch.tensor([r[k] for r in res], dtype=torch.float64) for k in ("lower_bound", "primal", "L")}
        return out | {k: torch.tensor([r[k] for r in res]) for k in ("iters", "trials", "restarts", "status")} | {"B": B}
    F, T = ctx.mlp_features(state["nodes"], state["Bp"], state["Bc"])
    return {"F": F, "T": T, "out": pr.mlp_forward(state["P"], F)}


def work(case):
    """Bytes and operations of one pass that the path cannot do without.  A relaxation reads the design once per
    evaluation (X^T times the dual vector; the iterate's own product touches only its support's columns), a batch does
    the two products with the design per iteration for all its nodes."""
    c, op = case, case["op"]
    if op == "prox":
        return {"bytes": c["p"] * (2 + 8 * 3), "flops": 20 * c["p"]}
    if op == "train":
        return {"bytes": c["rows"] * 20, "flops": c["rows"] * 6 * (8 * 64 + 64 * 64 + 64)}
    n, p, xb = c["n"], c["p"], n_bytes(c)
    rhs = 2 if c.get("loss") == LOGISTIC else 1
    if op == "solve":
        return {"bytes": c["evals"] * (xb + 8 * n * rhs + 8 * p * rhs), "flops": c["evals"] * 2 * n * p * rhs}
    if op == "bnb":
        return {"bytes": 55 * 16 * 8 * p * 200, "flops": 55 * 16 * 2 * p * 200}
    if op == "batch":
        if c["gram"]:
            return {"bytes": c["iters"] * 8 * p * p, "flops": c["iters"] * 2 * p * p * c["m"]}
        return {"bytes": c["iters"] * (xb + 8 * c["m"] * (n * rhs + p)), "flops": c["iters"] * 2 * n * p * c["m"] * (1 + rhs)}
    return {"bytes": 2 * xb + c["m"] * p * (8 + 8 + 16 + 4 + 4), "flops": c["m"] * (4 * n * p + p * 2 * (8 * 64 + 64 * 64))}


def n_bytes(c):
    return c["n"] * c["p"] * BYTES[c["dtype"]]


# ---------------------------------------------------------------- the same in 64 bits, plain torch
#
# Rows of every matrix below are nodes; st holds each node's status of each coordinate (0 free, 1 fixed to zero, 2
# fixed to one) and kb its number of free units.


def _huber(a, M):
    a = a.abs()
    return torch.where(a <= M, 0.5 * a * a, M * a - 0.5 * M * M) if math.isfinite(M) else 0.5 * a * a


def _x_top(a, kb):
    """The largest entries of each row in descending order, those past the row's kb set to zero."""
    kmax = max(1, int(kb.max()))
    t = a.topk(min(kmax, a.shape[1]), dim=1).values
    return torch.where(torch.arange(t.shape[1], device=a.device) < kb[:, None], t, 0.0)


def _x_gstar(w, st, kb, M):
    """sum of H_M over J1 plus the kb largest free values of H_M."""
    h = _huber(w, M)
    return torch.where(st == 2, h, 0.0).sum(1) + _x_top(torch.where(st == 0, h, 0.0), kb).sum(1)


def _x_g(x, st, kb):
    """0.5 sum omega^2 of Algorithm 1 plus the ridge on J1."""
    q = torch.where(st == 0, x.abs(), 0.0)
    theta = q.sum(1)
    top = _x_top(q, kb)
    K = kb[:, None].double()
    kept = torch.cat([torch.zeros_like(top[:, :1]), top.cumsum(1)], 1)  # kept[j]: sum of the j largest
    sq = torch.cat([torch.zeros_like(top[:, :1]), top.square().cumsum(1)], 1)
    j = torch.arange(kept.shape[1], device=x.device).double()[None]
    left = K - j
    bar = torch.where(left > 0, (theta[:, None] - kept) / left.clamp(min=1.0), math.inf)
    nxt = torch.cat([top, torch.zeros_like(top[:, :1])], 1)
    at = (bar >= nxt).double().argmax(1, keepdim=True)  # first j at which the mean of what is left covers the next
    free = sq.gather(1, at) + left.gather(1, at).clamp(min=0.0) * bar.gather(1, at).square()
    free = torch.where(K > 0, free, 0.0)[:, 0]
    return 0.5 * (free + torch.where(st == 2, x, 0.0).square().sum(1))


def _x_prox(v, rho, st, kb, M):
    """prox_{rho g_N}: magnitudes shifted by the threshold at which the fractions of the units add up to kb, by
    bisection and then the closed form for the sets found."""
    a = torch.where(st == 0, v.abs(), -1.0)
    rho = rho[:, None]
    K = kb[:, None].double()

    def width(t):
        return torch.clamp(t / rho, max=M)

    lo, hi = torch.zeros_like(K), a.max(1, keepdim=True).values.clamp(min=0.0)
    for _ in range(80):
        mid = 0.5 * (lo + hi)
        over = ((a - mid) / width(mid).clamp(min=1e-300)).clamp(0.0, 1.0).sum(1, keepdim=True) > K
        lo, hi = torch.where(over, mid, lo), torch.where(over, hi, mid)
    t = 0.5 * (lo + hi)
    block = (a > t) & (a <= t + width(t))
    head = (a > t + width(t)).sum(1, keepdim=True).double()
    nb, sb = block.sum(1, keepdim=True).double(), torch.where(block, a, 0.0).sum(1, keepdim=True)
    if math.isfinite(M):
        full = head + (sb - nb * rho * M) / M >= K
        root = torch.where(full, (sb - M * (K - head)) / nb, rho * sb / (K - head + rho * nb))
    else:
        root = rho * sb / (K - head + rho * nb)
    t = torch.where((nb > 0) & ((root - t).abs() <= 1e-9 * t), root, t)
    t = torch.where((a > 0).sum(1, keepdim=True) <= K, 0.0, t)
    r = torch.clamp(v.abs() / (1.0 + rho), max=M)
    r = torch.where(st == 0, torch.minimum(r, (v.abs() - t).clamp(min=0.0)), r)
    r = torch.where((st == 1) | ((st == 0) & (K <= 0)), 0.0, r)
    return torch.where(v < 0, -r, r)


def _x_norm2(X):
    """Largest eigenvalue of X X^T (X: (p, n)) by the Lanczos recurrence with full reorthogonalisation."""
    p = X.shape[0]
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    v = torch.randn(p, generator=g, device="cuda", dtype=torch.float64)
    V, al, be = [v / v.norm()], [], []
    last = 0.0
    for _ in range(min(p, 400)):
        w = X @ (X.T @ V[-1])
        al.append(float(w @ V[-1]))
        Q = torch.stack(V)
        for _ in range(2):
            w = w - Q.T @ (Q @ w)
        if len(al) % 8 == 0 or len(al) == p:
            T = torch.diag(torch.tensor(al, dtype=torch.float64))
            off = torch.tensor(be, dtype=torch.float64)
            T = T + torch.diag(off, 1) + torch.diag(off, -1)
            top = float(torch.linalg.eigvalsh(T)[-1])
            if top - last <= 1e-14 * top:
                return top
            last = top
        be.append(float(w.norm()))
        V.append(w / be[-1])
    return last


def _x_fista(X, y, logistic, st, kb, lam, M, L, tol, max_iter, linesearch, pair):
    """FISTA with the duality-gap restart (eta = e^3) on every row of st, fixed step 1/L or backtracking from L/16 by
    doublings up to L.  pair: stop on the gap of the current iterate and report it (batches), else report the best."""
    m = st.shape[0]
    dev = X.device
    lamc, eta = 2.0 * lam, math.exp(3.0)
    x = torch.zeros_like(st, dtype=torch.float64)
    u = torch.zeros(m, y.numel(), device=dev, dtype=torch.float64)
    xp, up = x.clone(), u.clone()
    Lk = torch.full((m,), L / 16.0 if linesearch else L, device=dev, dtype=torch.float64)
    t = torch.ones(m, device=dev, dtype=torch.float64)
    ref = torch.full((m,), math.inf, device=dev, dtype=torch.float64)
    lb, ub = torch.full_like(ref, -math.inf), torch.full_like(ref, math.inf)
    best, zbest = x.clone(), u.clone()
    live = torch.ones(m, dtype=torch.bool, device=dev)
    it = 0

    def dual(u):
        return y * torch.sigmoid(-y * u) if logistic else 2.0 * (y - u)

    while True:
        z = dual(u)
        w = z @ X.T
        if logistic:
            F = torch.nn.functional.softplus(-y * u).sum(1)
            a = torch.sigmoid(-y * u)
            conj = (a * torch.nn.functional.softplus(y * u) + (1 - a) * torch.nn.functional.softplus(-y * u)).sum(1)
        else:
            F = (y - u).square().sum(1)
            conj = z @ y - 0.25 * z.square().sum(1)
        phi = F + lamc * _x_g(x, st, kb)
        psi = conj - lamc * _x_gstar(w / lamc, st, kb, M)
        if pair:
            lb, ub = torch.where(live, psi, lb), torch.where(live, phi, ub)
            best[live] = x[live]
            stop = (phi - psi) <= 0.99 * tol * phi.abs()
        else:
            up_z, up_x = live & (psi > lb), live & (phi < ub)
            lb, ub = torch.where(up_z, psi, lb), torch.where(up_x, phi, ub)
            best[up_x], zbest[up_z] = x[up_x], z[up_z]
            stop = (ub - lb) <= tol * ub.abs()
        live = live & ~stop
        if it >= max_iter or not bool(live.any()):
            return lb, ub, best, zbest
        gap = phi - psi
        again = (gap <= ref / eta) if it else torch.ones_like(live)
        ref = torch.where(again, gap, ref)
        tn = 0.5 * (1.0 + (1.0 + 4.0 * t * t).sqrt())
        mom = torch.where(again, 0.0, (t - 1.0) / tn)
        t = torch.where(again, 1.0, tn)
        if linesearch:
            Lk = torch.where(again, L / 16.0, Lk)
        q = mom[:, None]
        yk, uk = x + q * (x - xp), (1.0 + q) * u - q * up
        grad = -(dual(uk) @ X.T)
        sel = live.clone()
        xn, un = x.clone(), u.clone()
        while bool(sel.any()):
            Ls = Lk[sel][:, None]
            xs = _x_prox(yk[sel] - grad[sel] / Ls, lamc / Ls[:, 0], st[sel], kb[sel], M)
            us = xs @ X
            xn[sel], un[sel] = xs, us
            if not linesearch:
                break
            du = us - uk[sel]
            if logistic:
                s, d = torch.sigmoid(-y * uk[sel]), -y * du
                D = (torch.log1p(s * torch.expm1(d)) - s * d).sum(1)
            else:
                D = du.square().sum(1)
            ok = (Ls[:, 0] >= L) | (D <= 0.5 * Ls[:, 0] * (xs - yk[sel]).square().sum(1))
            idx = sel.nonzero()[:, 0][~ok]
            Lk[idx] = torch.clamp(2.0 * Lk[idx], max=L)
            sel = torch.zeros_like(sel)
            sel[idx] = True
        xp, up, x, u = x, u, xn, un
        it += 1


def _x_status(c, nodes):
    st = torch.stack([torch.from_numpy(nd.status(c["p"])) for nd in nodes]).cuda()
    kb = torch.minimum(c["k"] - (st == 2).sum(1), (st == 0).sum(1))
    return st, kb


def _x_network(P, f):
    """The network on rows f, weights and activations as the FP32 parameters give them."""
    P = P.double()
    W1, b1, W2 = P[:512].view(64, 8), P[512:576], P[576:4672].view(64, 64)
    b2, w3, b3 = P[4672:4736], P[4736:4800], P[4800]
    a1 = (f @ W1.T + b1).clamp(min=0.0)
    a2 = (a1 @ W2.T + b2).clamp(min=0.0)
    return a1, a2, a2 @ w3 + b3


def exact(case, seed):
    c, op = case, case["op"]
    if op == "prox":
        v, w, st = _vector_inputs(c, seed)
        st = st[None]
        kb = torch.minimum(c["k"] - (st == 2).sum(1), (st == 0).sum(1))
        x = _x_prox(v[None], torch.tensor([c["rho"]], device="cuda", dtype=torch.float64), st, kb, c["M"])
        return {"x": x[0], "g": float(_x_g(x, st, kb)[0]), "gstar": float(_x_gstar(w[None], st, kb, c["M"])[0])}
    if op == "train":
        F, T = _train_rows(c, seed)
        P, m1, m2 = _network(seed)
        W2, w3 = P.double()[576:4672].view(64, 64), P.double()[4736:4800]
        rows, grad = c["rows"], torch.zeros(pr.MLP_NPARAM + 1, device="cuda", dtype=torch.float64)
        for i in range(0, rows, 1 << 17):
            f, tt = F[i:i + (1 << 17)].double(), T[i:i + (1 << 17)].double()
            a1, a2, out = _x_network(P, f)
            d = (out - tt) * (2.0 / rows)
            dz2 = torch.where(a2 > 0, d[:, None] * w3, 0.0)
            dz1 = torch.where(a1 > 0, dz2 @ W2, 0.0)
            grad += torch.cat([(dz1.T @ f).reshape(-1), dz1.sum(0), (dz2.T @ a1).reshape(-1), dz2.sum(0), a2.T @ d,
                               d.sum()[None], (out - tt).square().sum()[None] / rows])
        g, step = grad[:-1], 101
        n1, n2 = 0.9 * m1.double() + 0.1 * g, 0.999 * m2.double() + 0.001 * g * g
        new = P.double() - 1e-3 * (n1 / (1 - 0.9 ** step)) / ((n2 / (1 - 0.999 ** step)).sqrt() + 1e-8)
        return {"grad": grad, "params": new, "m1": n1, "m2": n2}
    if op == "bnb":
        return None
    X, y = _design(c, seed)
    X = X.double()
    logistic = c.get("loss") == LOGISTIC
    if op == "features":
        nodes = _nodes(c, seed)
        Bp, Bc = _parents(c, seed)
        u = Bp @ X
        w = (y * torch.sigmoid(-y * u) if logistic else 2.0 * (y - u)) @ X.T
        order = Bp.abs().sort(1).values
        rank = c["p"] - torch.searchsorted(order, Bp.abs().contiguous(), right=True)
        st, kb = _x_status(c, nodes)
        k = c["k"]
        one = torch.ones_like(Bp)
        cols = [Bp, w / w.abs().max(1, keepdim=True).values, rank / c["p"], (st == 2).double() - (st == 1).double(),
                c["lam"] * one, (st == 2).sum(1, keepdim=True) / k * one, (st == 1).sum(1, keepdim=True) / k * one,
                kb[:, None] / k * one]
        F = torch.stack(cols, 2).reshape(-1, 8)
        out = _x_network(_network(seed)[0], F.to(torch.bfloat16).double())[2]
        return {"F": F, "T": (Bc - Bp).reshape(-1), "out": out}
    if op == "batch":
        nodes = _nodes(c, seed)
    else:
        J0, J1 = _index_sets(seed, 5, c["p"], c["n0"], c["n1"])
        nodes = [pr.Node(c["k"], c["lam"], c["M"], J0=J0, J1=J1)]
    st, kb = _x_status(c, nodes)
    L = 1.01 * (0.25 if logistic else 2.0) * _x_norm2(X)
    if op == "batch":
        lb, ub, B, _ = _x_fista(X, y, logistic, st, kb, c["lam"], c["M"], L, 1e-6, c["iters"], True, True)
        return {"lower_bound": lb, "primal": ub, "L": None, "iters": None, "trials": None, "restarts": None,
                "status": None, "B": B}
    lb, ub, B, Z = _x_fista(X, y, logistic, st, kb, c["lam"], c["M"], L, c["tol"], c["max_iter"],
                            c["method"] == "linesearch", False)
    return {"lower_bound": float(lb), "primal": float(ub), "L": None, "iters": None, "trials": None, "restarts": None,
            "status": None, "beta": B[0], "zeta": Z[0]}
