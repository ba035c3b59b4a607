"""X x over the column list at the edges of its chunk planes (one plane, one
batch of 16, the largest count of one batch of 32 that is not full, two batches
of which the second is ragged, two full ones), and X^T r with one and two
right-hand sides on both sides of the lines between its two kernels."""
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
                                                ("f32", 4460, 3328, 52), ("f32", 2300, 5001, 64),
                                                # 1, 7, 13 and 16 + 8 columns per chunk: each size of the last round
                                                ("f32", 512, 16, 16), ("f32", 512, 100, 16), ("f64", 512, 200, 16),
                                                ("bf16", 512, 384, 16)])
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


# 10176 rows of right-hand sides fit in LDS; the other kernel serves p <= 4096 with two and p <= 10240 with one,
# so the second of each pair takes the LDS kernel and the last column of both may be alone in its pair
@pytest.mark.parametrize("storage,n,p", [("f32", 5088, 4096), ("f32", 5088, 4097), ("f32", 5092, 4099),
                                         ("f64", 2, 8193), ("bf16", 1032, 16390), ("f64", 130, 9007),
                                         ("bf16", 8, 4111)])
def test_two_right_hand_sides_by_kernel(dev, storage, n, p):
    import torch
    import paper_2603_01306_amd as pr
    X, g = _design(dev, storage, n, p, 5)
    y = torch.randn(n, generator=g, device=dev, dtype=torch.float64).sign()
    r = torch.randn(2, n, generator=g, device=dev, dtype=torch.float64)
    ctx = pr.Context(X, y, 1)
    h = ctx.gemv_t2(r[0].contiguous(), r[1].contiguous())
    for q in range(2):
        bound = 1e-13 * (X.double().abs() @ r[q].abs()) + 1e-300
        assert bool(((h[q] - X.double() @ r[q]).abs() <= bound).all())
    # one right-hand side sums every column in the same order, whichever kernel it takes
    assert torch.equal(h[0], ctx.gemv_t(r[0].contiguous()))
    ctx.close()


@pytest.mark.parametrize("storage,n,p", [("f32", 10176, 10240), ("f32", 10176, 10241), ("f32", 10180, 10243),
                                         ("f64", 64, 16390), ("bf16", 520, 20483)])
def test_one_right_hand_side_by_kernel(dev, storage, n, p):
    import torch
    import paper_2603_01306_amd as pr
    X, g = _design(dev, storage, n, p, 7)
    r = torch.randn(n, generator=g, device=dev, dtype=torch.float64)
    ctx = pr.Context(X, torch.randn(n, generator=g, device=dev, dtype=torch.float64), 0)
    h = ctx.gemv_t(r)
    for c in range(0, p, 2048):
        Xc = X[c:c + 2048].double()
        assert bool(((h[c:c + 2048] - Xc @ r).abs() <= 1e-13 * (Xc.abs() @ r.abs()) + 1e-300).all())
    ctx.close()


# the grids of the LDS kernel with two right-hand sides: equal rounds, or every resident workgroup with rounds of
# unequal length (the last one a single column), and their neighbours in the other kernel
@pytest.mark.parametrize("storage,n,p", [("bf16", 512, 16385), ("bf16", 2048, 16401), ("f32", 1024, 10241),
                                         ("f32", 1024, 8193), ("f32", 252, 16399), ("f64", 512, 14001),
                                         ("f64", 512, 18001), ("f32", 1024, 16385)])
def test_products_on_both_grids(dev, storage, n, p):
    import torch
    import paper_2603_01306_amd as pr
    X, g = _design(dev, storage, n, p, 11)
    r = torch.randn(2, n, generator=g, device=dev, dtype=torch.float64)
    ctx = pr.Context(X, torch.randn(n, generator=g, device=dev, dtype=torch.float64).sign(), 1)
    h = ctx.gemv_t2(r[0].contiguous(), r[1].contiguous())
    for q in range(2):
        assert torch.equal(h[q], ctx.gemv_t(r[q].contiguous()))
        for c in range(0, p, 4096):
            Xc = X[c:c + 4096].double()
            assert bool(((h[q][c:c + 4096] - Xc @ r[q]).abs() <= 1e-13 * (Xc.abs() @ r[q].abs()) + 1e-300).all())
    ctx.close()
