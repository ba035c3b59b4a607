"""Feature rows of many children at once (pr_mlp_features): supports of every
size against the oracle (one BF16 rounding of FP64 values, as the single-node
test), both losses, both routes (the batch's GEMMs for the images of all
nodes, two passes over X per node), more nodes than a context batches, and
malformed nodes."""
import numpy as np
import pytest

import oracle
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu

U = 2.0 ** -8  # unit roundoff of BF16


def _bf16(x):
    import torch
    return torch.from_numpy(np.asarray(x)).float().bfloat16().double().numpy()


@pytest.mark.parametrize("max_batch,m", [(1, 3), (70, 70), (40, 97)])  # 97: chunks of 40, 40 and 17
@pytest.mark.parametrize("loss", [0, 1])
def test_features_of_many_nodes(dev, max_batch, m, loss):
    import torch
    import paper_2603_01306_amd as pr
    print(f"features max_batch={max_batch} m={m} loss={loss}", flush=True)
    n, p, k = 256, 1152, 6
    rng = np.random.default_rng(100 * max_batch + loss)
    X = rng.standard_normal((p, n)).astype(np.float32)
    u = X[:4].astype(np.float64).sum(axis=0) + rng.standard_normal(n)
    y = u if loss == 0 else np.where(u >= 0, 1.0, -1.0)
    ctx = pr.Context(torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev), loss, max_batch=max_batch)
    Bp = np.zeros((m, p))
    nodes = []
    for i in range(m):
        nnz = (0, 1, 255, 256, 257, 1024, 1025, p)[i % 8]  # the rank kernel's workgroup and tile edges
        at = rng.permutation(p)
        Bp[i, at[:nnz]] = 0.02 * rng.standard_normal(nnz)
        Bp[i, at[:nnz // 2]] = np.round(Bp[i, at[:nnz // 2]], 2)  # ties and more zeros
        nodes.append(pr.Node(k, 0.3 + 0.01 * i, 2.0, J0=at[: i % 9], J1=at[20: 20 + i % (k + 1)]))
    Bc = Bp + rng.normal(0, 0.01, Bp.shape)
    F, T = ctx.mlp_features(nodes, torch.from_numpy(Bp).to(dev), torch.from_numpy(Bc).to(dev))
    assert torch.equal(F, ctx.mlp_features(nodes, torch.from_numpy(Bp).to(dev))[0])
    F = F.float().cpu().numpy().astype(np.float64).reshape(m, p, 8)
    assert np.array_equal(T.cpu().numpy().reshape(m, p), (Bc - Bp).astype(np.float32))
    X64 = X.astype(np.float64)
    for i, nd in enumerate(nodes):
        ui = Bp[i] @ X64
        z = 2.0 * (y - ui) if loss == 0 else y / (1.0 + np.exp(y * ui))
        ref = omlp.features(Bp[i], X64 @ z, nd.status(p), nd.lambda2, nd.k)
        assert np.all(np.abs(F[i] - _bf16(ref)) <= 2 * U * np.abs(ref) + 1e-30), i
        assert np.array_equal(F[i, :, 2], _bf16(ref[:, 2]))  # ranks are counts
    with pytest.raises(pr.PrError):
        ctx.mlp_features([nodes[0], pr.Node(k, 0.3, 2.0, J0=[p])], torch.from_numpy(Bp[:2]).to(dev))
    ctx.close()


@pytest.mark.parametrize("p", [1, 257, 1152, 4096, 4097])
def test_features_of_one_node(dev, p):
    """One node's rows on both sides of the size from which its ranks get a
    launch of their own (4096 | 4097), supports of every size around the list's
    tiles: against the oracle as above, ranks exactly."""
    import torch
    import paper_2603_01306_amd as pr
    print(f"features of one node p={p}", flush=True)
    n, k = 8, 6
    rng = np.random.default_rng(p)
    X = rng.standard_normal((p, n)).astype(np.float32)
    y = X[:4].astype(np.float64).sum(axis=0) + rng.standard_normal(n)
    ctx = pr.Context(torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev), 0)
    X64 = X.astype(np.float64)
    for nnz in sorted({min(v, p) for v in (0, 1, 255, 1023, 1024, 1025, p)}):
        at = rng.permutation(p)
        b = np.zeros(p)
        b[at[:nnz]] = np.round(0.02 * rng.standard_normal(nnz), 3)  # ties and more zeros
        nd = pr.Node(k, 0.3, 2.0, J0=at[: min(3, p - 1)], J1=at[3:5])
        F = ctx.mlp_features([nd], torch.from_numpy(b[None]).to(dev))[0].float().cpu().numpy().astype(np.float64)
        ref = omlp.features(b, X64 @ (2.0 * (y - b @ X64)), nd.status(p), nd.lambda2, nd.k)
        assert np.all(np.abs(F - _bf16(ref)) <= 2 * U * np.abs(ref) + 1e-30), nnz
        assert np.array_equal(F[:, 2], _bf16(ref[:, 2])), nnz
    ctx.close()
