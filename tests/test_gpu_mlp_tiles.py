"""Edges of the network kernels' tiles (16 samples per tile, 16 x 16 gradient
tiles over groups of four samples, sixteen groups in flight) and arrays that
start off a 16-byte boundary, against the FP64 oracle.  Bars as for the other
sizes: FP32 sums of 16 and 64 products, 1e-5 relative."""

import sys

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "offset4"])
@pytest.mark.parametrize("n", [1, 4, 15, 16, 17, 65, 1023, 1025])
def test_tile_edges_match_oracle(n, offset):
    import torch
    from paper_2410_21607_amd import api
    print("mlp tiles", n, offset, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(100 + n)
    p = (rng.standard_normal(mlp.N_PARAM) * 0.3).astype(np.float32)
    x = rng.standard_normal((n, 16)).astype(np.float32)
    y = rng.integers(0, 3, size=n).astype(np.int8)

    def dev(a):
        t = torch.empty(a.size + 4, dtype=torch.float32, device="cuda")[offset:offset + a.size]
        t.copy_(torch.as_tensor(a.reshape(-1)))
        return t

    P, X, Y = dev(p), dev(x).view(n, 16), torch.as_tensor(y).cuda()
    # guard values behind every output: nothing may be written past the end
    logits = torch.full((n * 3 + 8,), 7.0, device="cuda")
    api.mlp_forward(P, X, logits[:n * 3])
    work = torch.full((n * api.MLP_WORK + 8,), 7.0, device="cuda")
    grad = torch.full((mlp.N_PARAM + 8,), 7.0, device="cuda")
    loss = torch.zeros(1, device="cuda")
    w = work[offset:offset + n * api.MLP_WORK]
    api.mlp_backward(P, X, Y, None, w, grad[:mlp.N_PARAM], loss)
    torch.cuda.synchronize()
    assert torch.all(logits[n * 3:] == 7.0) and torch.all(grad[mlp.N_PARAM:] == 7.0)
    assert torch.all(work[offset + n * api.MLP_WORK:] == 7.0) and torch.all(work[:offset] == 7.0)
    z, _, _ = mlp.forward(p.astype(np.float64), x.astype(np.float64))
    got = logits[:n * 3].cpu().numpy().reshape(n, 3)
    assert np.max(np.abs(got - z)) <= 1e-5 * max(1.0, np.max(np.abs(z)))
    L, g = mlp.gradient(p.astype(np.float64), x.astype(np.float64), y.astype(np.int64))
    gg = grad[:mlp.N_PARAM].cpu().numpy().astype(np.float64)
    assert abs(float(loss.item()) - L) <= 1e-5 * max(1.0, L)
    for name, _ in mlp.SHAPES:
        a, b = mlp.unflatten(gg)[name], mlp.unflatten(g)[name]
        assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(b) + 1e-9, name
