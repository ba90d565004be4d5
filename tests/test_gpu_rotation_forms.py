"""Rotations taken out of their larger entry (one fused multiply-add per
component, the entries' product put back by the pass's scale): both forms of RX
and RY, at angles around the change of form and at the entries' zeros, next to
controlled rotations, and enough of them in one pass for the scale in between;
against the oracle. Each gate rounds an amplitude (at most 1) a few times:
m gates are within 4 m 2^-24 of the oracle in complex64, 4 m 2^-53 in
complex128, and the compiled pass equals the interpreted one bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu

ANGLES = [0.0, 1e-9, 0.3, np.pi / 2 - 1e-7, np.pi / 2, np.pi / 2 + 1e-7, 2.0, np.pi, 4.0, 3 * np.pi / 2, 5.5, 2 * np.pi, -0.7, 7.0]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,reps", [(6, 1), (13, 1), (15, 1), (7, 12)])
def test_rotations_out_of_their_larger_entry(n, reps, dtype, monkeypatch):
    rng = np.random.default_rng([n, reps])
    rows = []
    for _ in range(reps):
        for a in ANGLES:
            for kind in ("RX", "RY"):
                q = int(rng.integers(0, n))
                rows.append((kind, q, -1, float(a)))
                if rng.random() < 0.3:
                    rows.append((kind, q, (q + 1) % n, float(a)))
                if rng.random() < 0.3:
                    rows.append(("H", (q + 2) % n, -1, 0.0))
    g = W.gates_from_tuples(rows)
    a = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    a = (a / np.linalg.norm(a)).astype(np.complex64 if dtype == "c64" else np.complex128)
    out = []
    for jit in ("1", "0"):
        monkeypatch.setenv("SV_JIT", jit)
        s = sv.StateVector(n, dtype)
        try:
            print(f"case rotations n={n} reps={reps} {dtype} jit={jit}", flush=True)
            s.set_state(a)
            s.apply(g)
            out.append(s.state())
        finally:
            s.close()
    assert np.array_equal(out[0], out[1])
    want = oracle.apply(n, g, a.astype(np.complex128))
    eps = 2.0 ** -24 if dtype == "c64" else 2.0 ** -53
    assert np.max(np.abs(out[0] - want)) <= 4 * len(g) * eps
