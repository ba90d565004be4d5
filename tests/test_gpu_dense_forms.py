"""Dense gates whose matrix has zero halves (RX, RY and the like) against the
plain sweep, bit for bit, and the FP64 oracle (80 gates of at most 8 roundings
of 2^-24 on amplitudes below 1: 4e-5 in complex64, 1e-12 in complex128)."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"c64": 4e-5, "c128": 1e-12}


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("jit", ["1", "0"])
def test_real_and_cross_matrices(dtype, jit, monkeypatch):
    """Dense gates with zero halves, controlled by every class of bit: the same bits as the plain sweep's full product."""
    monkeypatch.setenv("SV_JIT", jit)
    n = 13
    rng = np.random.default_rng(9)
    rows = []
    for kind in ("RX", "RY", "Y", "RX", "RY"):
        for q in range(n):
            rows.append((kind, q, int((q + 1 + rng.integers(0, n - 1)) % n) if rng.random() < 0.5 else -1, float(rng.random() * 6)))
    g = W.gates_from_tuples(rows)
    u2 = np.zeros(4, dtype=W.GATE_DTYPE)
    u2["op"], u2["target2"], u2["control"] = W.OP_U2, -1, -1
    u2["target"] = [0, 5, 12, 7]
    u2["control"][2:] = [3, 11]
    c, sn = np.cos(0.7), np.sin(0.7)
    u2["u"][0] = [c, 0, sn, 0, sn, 0, -c, 0]     # real
    u2["u"][1] = [c, 0, 0, sn, 0, sn, c, 0]      # real diagonal, imaginary off it
    u2["u"][2] = [0, c, sn, 0, -sn, 0, 0, -c]    # imaginary diagonal: the full product
    u2["u"][3] = u2["u"][1]
    g = np.concatenate([g, u2, g[::-1]])
    out = []
    for sched in (sv.schedule(fuse_k=0, swap_policy="lookahead"), sv.schedule("plain")):  # gates in list order
        s = sv.StateVector(n, dtype)
        try:
            s.apply(g, sched)
            out.append(s.state())
        finally:
            s.close()
    assert np.array_equal(out[0], out[1])
    assert np.max(np.abs(out[0] - oracle.apply(n, g))) <= TOL[dtype]
