"""Circuits applied again on one handle: what the handle keeps of a plan must
never be used for another circuit, layout, schedule or mode. Every result is
compared with the FP64 oracle's (80 gates of at most 8 roundings of 2^-24 on
amplitudes below 1: 4e-5 in complex64, 1e-12 in complex128)."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"c64": 4e-5, "c128": 1e-12}


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_alternating_circuits_layouts_and_modes(dtype, monkeypatch):
    n = 12
    rng = np.random.default_rng(77)
    base = W.random_mixed_circuit(n, 40, rng, with_swap=True)   # SWAPs: the layout moves on with every call
    circuits = [base]
    for i in range(10):                                          # more than a handle keeps, equal but for one entry
        g = base.copy()
        j = int(np.flatnonzero((g["op"] >= W.OP_RX) & (g["op"] <= W.OP_P))[i % 5])
        g[j]["theta"] += 0.1 + i
        circuits.append(g)
    circuits.append(base[:-1])
    scheds = [None, sv.schedule(fuse_k=0), sv.schedule(block_qubits=8), sv.schedule("plain")]
    want = np.zeros(1 << n, dtype=np.complex128)
    want[0] = 1
    s = sv.StateVector(n, dtype)
    try:
        for step, k in enumerate(rng.integers(0, len(circuits), size=60).tolist()):
            monkeypatch.setenv("SV_JIT", "0" if step % 3 == 2 else "1")
            if step % 20 == 19:
                s.reset()
                want[:] = 0
                want[0] = 1
            print(f"case prepared {dtype} step={step} circuit={k}", flush=True)
            s.apply(circuits[k], scheds[step % 4])
            want = oracle.apply(n, circuits[k], want)
            if step % 7 == 6:
                s.set_state(want)                                # keeps rounding from adding up
                want = want.astype(np.complex64).astype(np.complex128) if dtype == "c64" else want
            assert np.max(np.abs(s.state() - want)) <= TOL[dtype] * 2, step
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [3, 10, 11, 13, 18, 19, 20, 21, 22, 23])
def test_default_schedule_by_size(n, dtype):
    """The default blocks on both sides of each change of size, compiled and interpreted alike."""
    rng = np.random.default_rng([n, 8])
    g = W.random_mixed_circuit(n, 60, rng)
    want = oracle.apply(n, g)
    states = []
    for jit in ("1", "0"):
        with pytest.MonkeyPatch.context() as mp:
            mp.setenv("SV_JIT", jit)
            s = sv.StateVector(n, dtype)
            try:
                print(f"case by size n={n} {dtype} jit={jit}", flush=True)
                s.apply(g)
                states.append(s.state())
            finally:
                s.close()
        assert np.max(np.abs(states[-1] - want)) <= TOL[dtype]
    assert np.array_equal(states[0], states[1])
