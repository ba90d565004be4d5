"""Programs of the default schedule (block, tile and pins by size) on the CPU:
the planner's passes emulated op by op against the FP64 oracle, at the sizes
where the rule changes, and its pass counts at sizes too large to emulate."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W
from test_plan_emulator import run


@pytest.mark.parametrize("fuse", [0, 1, 5])
@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [1, 2, 4, 5, 6, 9, 10, 11, 12, 13, 15])
def test_programs_by_size(n, dtype, fuse):
    rng = np.random.default_rng([n, 6])
    g = W.random_mixed_circuit(n, 80, rng)
    psi0 = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi0 /= np.linalg.norm(psi0)
    got, _ = run(n, g, psi0, dtype=dtype, l=0, logr=0, policy=2, pin=-1, fuse=fuse)
    # the emulator computes in FP64; 80 gates of a few roundings each
    assert np.max(np.abs(got - oracle.apply(n, g, psi0))) < 1e-12


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [8, 17, 18, 19, 20, 21, 22, 23, 24, 25, 28, 32])
def test_pass_counts_by_size(n, dtype):
    """In complex64, and from 22 qubits on in complex128, the blocks are the
    largest, and choosing the pins never costs more passes than the longest
    runs."""
    rng = np.random.default_rng([n, 7])
    for g in (W.qpe_gates(n, 0.3), W.random_circuit(n, 200, rng)):
        auto = sv.sv_plan(n, dtype, g, None)
        assert auto["gates"] == int(np.sum(g["op"] != W.OP_SWAP))
        if n >= 23 or (dtype == "c64" and n >= 14):
            largest = dict(block_qubits=14 if dtype == "c64" else 13, reg_qubits=5 if dtype == "c64" else 4)
            longest = sv.sv_plan(n, dtype, g, sv.schedule(pin_qubits=5 if dtype == "c64" else 4, **largest))
            assert auto["passes"] <= longest["passes"]
            assert auto["block_qubits"] == largest["block_qubits"]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [8, 16, 18, 20, 23, 24, 26, 28, 31])
def test_written_out_default(n, dtype):
    """The default that tuned schedules are compared with plans as the default does."""
    from paper_2605_15098_amd import costmodel
    for g in (W.qpe_gates(n, 0.3), W.random_circuit(n, 200, np.random.default_rng([n, 8]))):
        assert sv.sv_plan(n, dtype, g, costmodel.default_schedule(n, dtype, g)) == sv.sv_plan(n, dtype, g, None)
