"""The network kernels at the edges of their tiles of 16 samples, and with more
tiles than the gradient kernel has work-groups (128), against the FP64 oracle.
Bars as for the other network tests: 1e-5 relative for predictions and loss,
1e-4 for gradients (FP32 products and sums of at most 2049 samples)."""
import numpy as np
import pytest

from oracle import mlp
from paper_2605_15098_amd import sv
from test_gpu_mlp import dev, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("in_dim", [1, 15, 16, 17, 32])
@pytest.mark.parametrize("batch", [1, 15, 16, 17, 129, 2048, 2049])
def test_tiles(in_dim, batch):
    import torch
    p, x, norm, t = inputs(in_dim, batch, 5 + batch)
    print(f"case mlp tiles in={in_dim} batch={batch}", flush=True)
    y, grad, loss = torch.zeros(batch, device="cuda"), torch.zeros(len(p), device="cuda"), torch.zeros(1, device="cuda")
    ws = torch.full((sv.sv_mlp_workspace_bytes(in_dim, batch) // 4,), 7.0, device="cuda")
    sv.sv_mlp_forward(dev(p), in_dim, dev(norm), dev(x), batch, y)
    sv.sv_mlp_grad(dev(p), in_dim, dev(norm), dev(x), dev(t), batch, grad, loss, ws)
    want = mlp.forward(p.astype(np.float64), norm, x)
    assert np.all(np.abs(y.cpu().numpy() - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))
    lw, gw = mlp.loss_and_grad(p.astype(np.float64), norm, x, t)
    got = grad.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - gw)) <= 1e-4 * np.max(np.abs(gw))
    assert abs(float(loss.item()) - lw) <= 1e-5 * max(1.0, lw)
