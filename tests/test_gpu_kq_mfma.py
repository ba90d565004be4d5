"""GPU parity of k-qubit unitaries (k = 4..6) on the matrix cores against the
FP64 oracle: the smallest states that take them (32 groups) and those just
below, targets on the lowest, highest and mixed qubits in any order, controls.

An output is a dot product of 2 * 2^k real terms of a unit row with a state of
norm 1 (sum of magnitudes at most sqrt 2), plus the rounding of the matrix
itself: (2^(k+1) + 2) * eps * sqrt(2) bounds its error.
"""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv

pytestmark = pytest.mark.gpu

EPS = {"c64": 2.0 ** -24, "c128": 2.0 ** -53}


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("k", [4, 5, 6])
@pytest.mark.parametrize("extra", [3, 4, 5, 6, 10])
def test_unitary(k, extra, dtype):
    n = k + extra
    rng = np.random.default_rng([k, extra])
    q = list(range(n))
    picks = [q[:k], q[-k:], q[:k][::-1], [int(x) for x in rng.choice(n, size=k, replace=False)]]
    s = sv.StateVector(n, dtype)
    try:
        a = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
        a = (a / np.linalg.norm(a)).astype(np.complex64 if dtype == "c64" else np.complex128)
        for targets in picks:
            free = [x for x in q if x not in targets]
            for controls in ([], free[:1], [int(x) for x in rng.choice(free, size=min(3, len(free)), replace=False)]):
                d = 1 << k
                u, r = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
                print(f"case kq n={n} {dtype} targets={targets} controls={controls}", flush=True)
                s.set_state(a)
                g = [("U", targets, controls, u)]
                s.apply_ex(g)
                want = oracle.apply_ex(n, g, a.astype(np.complex128))
                err = np.max(np.abs(s.state().astype(np.complex128) - want))
                assert err <= (2 ** (k + 1) + 2) * EPS[dtype] * 2 ** 0.5, (targets, controls, err)
    finally:
        s.close()
