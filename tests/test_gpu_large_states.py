"""GPU: sizes near the limits of launches and counters. States of 64 GiB and
more, where a thread per unit of work is more threads than one launch may have
(2^32), and batches of the cost-model network up to the largest int."""
import numpy as np
import pytest

from oracle import mlp
from oracle import qpe as cf
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu


class Wrapped:
    """A handle on a buffer of ones that starts `skip` real numbers into its allocation."""

    def __init__(self, n, dtype, skip=0):
        import torch
        torch.cuda.empty_cache()
        self.n, self.dtype = n, dtype
        self.buf = torch.full(((2 << n) + 2 * skip,), 1.0, dtype=torch.float32 if dtype == "c64" else torch.float64, device="cuda")
        size = self.buf.element_size()
        self.h = sv.sv_wrap(n, dtype, self.buf.data_ptr() + skip * size, (2 << n) * size)

    def close(self):
        import torch
        sv.sv_destroy(self.h)
        self.buf = None
        torch.cuda.empty_cache()


@pytest.mark.parametrize("dtype,n,skip", [("c64", 32, 2), ("c64", 33, 0), ("c128", 32, 0)])
def test_reset_and_phase_estimation(dtype, n, skip):
    print(f"case reset n={n} {dtype} skip={skip}", flush=True)
    w = Wrapped(n, dtype, skip)
    try:
        sv.sv_reset(w.h)
        # every other amplitude would add 2 to the sum of squares
        assert sv.sv_norm(w.h) == 1.0
        for off in (0, 1 << (n - 1), (1 << n) - 4):
            assert np.array_equal(sv.sv_state_range(w.h, off, 4, dtype), np.eye(4)[0] if off == 0 else np.zeros(4))
        if skip:
            assert w.buf[:skip].tolist() == [1.0] * skip and w.buf[-skip:].tolist() == [1.0] * skip
        phi = W.phi_for_seed(n)
        sv.sv_apply_circuit(w.h, W.qpe_gates(n, phi))
        m, _, p = sv.sv_qpe_readout(w.h, n - 1)
        want = cf.qpe_argmax(n - 1, phi)
        # the project's bounds on an amplitude, twice for its square
        assert m == want and abs(p - cf.qpe_probabilities(n - 1, phi, [want])[0]) <= (2e-12 if dtype == "c128" else 4e-5)
    finally:
        w.close()


@pytest.mark.parametrize("what,n", [("unitary", 33), ("plain", 34)])
def test_gates_in_more_than_one_launch(what, n):
    """Amplitudes on both sides of where a sweep over complex64 amplitudes splits: a dense 2x2 unitary
    from 2^33 amplitudes on, an RZ without control in a plain circuit from 2^34 on."""
    print(f"case split {what} n={n}", flush=True)
    w = Wrapped(n, "c64")
    try:
        sv.sv_reset(w.h)
        half = 1 << (n - 1)
        for at, a in ((0, [0, 0, 0.6, 0]), (half, [0, 0, 0, 0.8j])):
            sv.sv_set_state_range(w.h, at, np.array(a, dtype=np.complex64))
        th = 0.7
        c, s, e = np.cos(th / 2), np.sin(th / 2), np.exp(0.5j * th)
        if what == "unitary":
            sv.sv_apply_circuit_ex(w.h, [("U", [0], [], np.array([[c, -s], [s, c]], dtype=complex))])
            want = ((0, [0, 0, 0.6 * c, 0.6 * s]), (half, [0, 0, -0.8j * s, 0.8j * c]))
        else:
            sv.sv_apply_circuit(w.h, W.gates_from_tuples([("RZ", 0, -1, th)]), sv.schedule("plain"))
            want = ((0, [0, 0, 0.6 / e, 0]), (half, [0, 0, 0, 0.8j * e]))
        for at, a in want:
            # two FP32 roundings of each product of entries rounded once
            assert np.max(np.abs(sv.sv_state_range(w.h, at, 4, "c64") - np.array(a))) <= 4 * 2.0 ** -24
        assert abs(sv.sv_norm(w.h) - 1.0) <= 16 * 2.0 ** -24
    finally:
        w.close()


def test_network_on_the_largest_batch():
    """2^31 - 1 samples of one input: predictions at both ends and around the last 2^14 samples, where an int
    that counts samples in steps of the grid wraps; the gradient of a network that predicts 1/2 everywhere."""
    import torch
    batch = (1 << 31) - 1
    rng = np.random.default_rng(9)
    p = rng.normal(size=sv.sv_mlp_param_count(1)).astype(np.float32) * 0.3
    x, y = torch.empty(batch, device="cuda"), torch.full((batch,), np.nan, device="cuda")
    x.uniform_(-2.0, 2.0)
    print("case network forward", flush=True)
    sv.sv_mlp_forward(torch.tensor(p, device="cuda"), 1, None, x, batch, y)
    norm = np.array([0.0, 1.0])
    for at in (0, batch - (1 << 14) - 512, batch - 1024):
        want = mlp.forward(p.astype(np.float64), norm, x[at:at + 1024].cpu().numpy().astype(np.float64).reshape(-1, 1))
        assert np.all(np.abs(y[at:at + 1024].cpu().numpy() - want) <= 1e-5 * np.maximum(1.0, np.abs(want)))
    assert not bool(torch.isnan(y).any())
    p[:] = 0.0
    p[-1] = 0.5
    y.zero_()
    grad, loss = torch.zeros(len(p), device="cuda"), torch.zeros(1, device="cuda")
    ws = torch.full((sv.sv_mlp_workspace_bytes(1, batch) // 4,), 7.0, device="cuda")
    print("case network gradient", flush=True)
    sv.sv_mlp_grad(torch.tensor(p, device="cuda"), 1, None, x, y, batch, grad, loss, ws)
    # sums of equal powers of two: exact but for the last, incomplete tile
    assert abs(float(loss.item()) - 0.25) <= 1e-6 and abs(float(grad[-1].item()) - 1.0) <= 1e-6
    assert not bool(grad[:-1].any())
