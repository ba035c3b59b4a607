"""Kernels whose workgroups share one vector, when the last workgroup gives up
its first wait (a test switch of the context): the launches end, the call fails
with PR_EDEVICE, and the context gives its former results once the switch is
off."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _context(dev, p, n=32, loss=0):
    import torch
    import paper_2603_01306_amd as pr
    rng = np.random.default_rng(p)
    X = rng.standard_normal((p, n)).astype(np.float32)
    y = X[:4].astype(np.float64).sum(axis=0)
    y = y if loss == 0 else np.where(y >= 0, 1.0, -1.0)
    beta = torch.from_numpy(0.01 * rng.standard_normal(p)).to(dev)
    beta[1] = 0.0
    return pr.Context(torch.from_numpy(X).to(dev), torch.from_numpy(y).to(dev), loss), beta


def _edevice(fn):
    import paper_2603_01306_amd as pr
    with pytest.raises(pr.PrError) as e:
        fn()
    assert "-3" in str(e.value)


@pytest.mark.parametrize("p", [4097, 20000, 262145])
def test_lost_exchange_in_bounds_and_warm_start(dev, p):
    import torch
    import paper_2603_01306_amd as pr
    print(f"lost exchange p={p}", flush=True)
    ctx, beta = _context(dev, p)
    node = pr.Node(5, 0.5, float("inf"), J0=[1], J1=[2])
    calls = (lambda: ctx.dual_bound(node, beta=beta), lambda: ctx.mlp_warm_start([node], None, beta[None]))
    good = [c() for c in calls]
    ctx.set_debug(pr.DEBUG_LOSE_EXCHANGE)
    for c in calls:
        _edevice(c)
    ctx.set_debug(0)
    again = [c() for c in calls]
    assert again[0] == good[0] and np.isfinite(good[0]).all()
    assert torch.equal(again[1][0], good[1][0]) and np.array_equal(again[1][2], good[1][2])
    ctx.close()


def test_lost_exchange_in_the_gram_certificate(dev):
    import torch
    import paper_2603_01306_amd as pr
    print("lost exchange gram", flush=True)
    ctx, _ = _context(dev, 4224)
    ctx.enable_gram()
    node = pr.Node(5, 2.0, 2.0)
    good = ctx.solve(node, want_zeta=True, max_iter=40)
    ctx.set_debug(pr.DEBUG_LOSE_EXCHANGE)
    _edevice(lambda: ctx.solve(node, want_zeta=True, max_iter=40))
    ctx.set_debug(0)
    again = ctx.solve(node, want_zeta=True, max_iter=40)
    assert again["lower_bound"] == good["lower_bound"] and torch.equal(again["zeta"], good["zeta"])
    ctx.close()


@pytest.mark.parametrize("p,loss", [(16385, 0), (20000, 1), (262145, 1)])
def test_lost_exchange_in_the_solve(dev, p, loss):
    """beta = 0: the start's only exchange is lost by the last workgroup alone,
    the first one completes."""
    import torch
    import paper_2603_01306_amd as pr
    print(f"lost exchange solve p={p} loss={loss}", flush=True)
    ctx, beta = _context(dev, p, n=16, loss=loss)
    node = pr.Node(5, 1.0, 2.0)
    kw = dict(max_iter=12, rel_gap_tol=0.0, L=50.0)
    good = [ctx.solve(node, beta0=b0, **kw) for b0 in (None, beta)]
    ctx.set_debug(pr.DEBUG_LOSE_EXCHANGE)
    for b0 in (None, beta):
        _edevice(lambda: ctx.solve(node, beta0=b0, **kw))
    ctx.set_debug(0)
    for b0, g in zip((None, beta), good):
        again = ctx.solve(node, beta0=b0, **kw)
        assert (again["lower_bound"], again["primal"]) == (g["lower_bound"], g["primal"])
        assert torch.equal(again["beta"], g["beta"])
    ctx.close()
