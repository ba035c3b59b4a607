"""X x over the column list at the edges of its chunk planes: one plane, one
batch of 16, the largest count of one batch of 32 that is not full, two batches
of which the second is ragged, two full ones."""
import pytest

pytestmark = pytest.mark.gpu


def _design(dev, storage, n, p, seed):
    import torch
    g = torch.Generator(device=dev).manual_seed(seed)
    X = torch.randn(p, n, generator=g, device=dev, dtype=torch.float64)
    return X.to({"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}[storage]), g


# row blocks hold 256 x 16 bytes of a column; the planes: p where it is below 16, else 16, else with 64 columns
# per chunk at least as many as give every compute unit a workgroup, 64 at most
@pytest.mark.parametrize("storage,n,p,planes", [("f64", 2, 1, 1), ("f32", 64, 15, 15), ("f32", 1024, 4095, 16),
                                                ("bf16", 16384, 2047, 16), ("f64", 4608, 1920, 29),
                                                ("f32", 4460, 3328, 52), ("f32", 2300, 5001, 64)])
def test_column_list_product_at_plane_counts(dev, storage, n, p, planes):
    import torch
    import paper_2603_01306_amd as pr
    X, g = _design(dev, storage, n, p, 3 + planes)
    y = torch.randn(n, generator=g, device=dev, dtype=torch.float64)
    b = torch.randn(p, generator=g, device=dev, dtype=torch.float64)
    ctx = pr.Context(X, y, 0)
    u = ctx.gemv(b)
    assert torch.equal(u, ctx.gemv(b))
    # both sides sum exact FP64 products of at most p terms in some order
    bound = 1e-13 * (X.double().abs().T @ b.abs()) + 1e-300
    assert bool(((u - X.double().T @ b).abs() <= bound).all())
    ctx.close()
