"""Gradient of the warm-start network at the edges of its row tiles: one row,
one row less and more than a wave's 32 and a workgroup's 128, the largest count
with one tile per workgroup and the first with two; rows past the end hold NaN."""
import numpy as np
import pytest

from oracle import mlp as omlp
from test_gpu_mlp import _bf16, _dev, _forward_bound, _grad_error_bound, _pr, _rand_params, _rand_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 31, 33, 127, 128, 129, 65536, 65537])
def test_gradient_at_tile_edges(dev, rows):
    import torch
    pr = _pr()
    P = _rand_params(21 + rows, bf16_weights=False)
    F, T = _rand_rows(23 + rows, rows)
    Fd = torch.full((rows + 200, omlp.NF), float("nan"), dtype=torch.bfloat16, device=dev)
    Td = torch.full((rows + 200,), float("nan"), dtype=torch.float32, device=dev)
    Fd[:rows] = _dev(F, torch.float32).to(torch.bfloat16)
    Td[:rows] = _dev(T, torch.float32)
    Pb = P.copy()
    Pb[omlp.OFF_W1:omlp.OFF_B1] = _bf16(P[omlp.OFF_W1:omlp.OFF_B1])
    Pb[omlp.OFF_W2:omlp.OFF_B2] = _bf16(P[omlp.OFF_W2:omlp.OFF_B2])
    Pd = _dev(P, torch.float32)
    g = pr.mlp_grad(Pd, Fd[:rows], Td[:rows])
    assert torch.equal(g, pr.mlp_grad(Pd, Fd[:rows], Td[:rows]))
    g = g.cpu().numpy().astype(np.float64)
    loss, ref = omlp.loss_grad(Pb, F, T)
    assert np.all(np.abs(g[:-1] - ref) <= _grad_error_bound(Pb, F, T))
    # each output is within the forward's bound e, so each (out - T)^2 within (2 |out - T| + e) e
    d, e = np.abs(omlp.forward(Pb, F) - T), _forward_bound(Pb, F)
    assert abs(g[-1] - loss) <= np.mean((2.0 * d + e) * e) + 1e-6 * loss
