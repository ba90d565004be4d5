"""The phase readout at the edges of its chunks of 2^11 entries."""
import numpy as np
import pytest

from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 3, 8, 10, 11, 12, 13, 16, 21])
def test_phase_readout(n, dtype):
    """Index and value of the largest marginal entry, every complement up to 4 qubits, in two layouts, with ties."""
    rng = np.random.default_rng([n, 4])
    s = sv.StateVector(n, dtype)
    try:
        for swap in (False, True):
            a = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
            a[rng.integers(0, 1 << n)] *= 6
            a = (a / np.linalg.norm(a)).astype(np.complex64 if dtype == "c64" else np.complex128)
            if swap:
                s.apply(W.gates_from_tuples([("SWAP", q, -1, 0.0, n - 1 - q) for q in range(n // 2)]))
            for state in (a, np.full(1 << n, 2.0 ** (-n / 2), dtype=a.dtype), np.zeros(1 << n, dtype=a.dtype)):
                s.set_state(state)
                for t in range(max(1, n - 4), n + 1):
                    p = (np.abs(state.astype(np.complex128)) ** 2).reshape(1 << (n - t), 1 << t).sum(axis=0)
                    print(f"case readout n={n} {dtype} t={t} swap={swap}", flush=True)
                    for call in (sv.sv_qpe_readout, sv.sv_qpe_readout_noalloc):
                        m, phi, pm = call(s.h, t)
                        assert abs(pm - p.max()) <= 1e-14 and phi == m / 2.0 ** t
                        assert m == int(np.argmax(p)) or (m < 1 << t and abs(p[m] - p.max()) <= 1e-16)
    finally:
        s.close()
