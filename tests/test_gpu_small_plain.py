"""Plain circuits of small states as one launch: the same bits as a launch per
gate (what kernel timing asks for), at the smallest states, around a wave, a
work-group's threads, and the largest that fit in LDS, with one and two gates
as well."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [1, 2, 5, 6, 7, 8, 10, 11, 12, 13, 14, 15])
def test_one_launch_equals_launch_per_gate(n, dtype):
    rng = np.random.default_rng([n, 3])
    a = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    a = (a / np.linalg.norm(a)).astype(np.complex64 if dtype == "c64" else np.complex128)
    for depth in (1, 2, 70):
        g = W.random_mixed_circuit(n, depth, rng)
        out = []
        for timing in (False, True):
            s = sv.StateVector(n, dtype)
            try:
                print(f"case small plain n={n} {dtype} depth={depth} timing={timing}", flush=True)
                sv.sv_set_kernel_timing(s.h, timing)
                s.set_state(a)
                s.apply(g, sv.schedule("plain"))
                out.append(s.state())
                gates = int(np.sum(g["op"] != W.OP_SWAP))
                assert s.stats()["passes"] == gates
                if timing:
                    assert s.stats()["kernel_launches"][0] == gates
            finally:
                s.close()
        assert np.array_equal(out[0], out[1])
        want = oracle.apply(n, g, a.astype(np.complex128))
        assert np.max(np.abs(out[0] - want)) <= (4e-5 if dtype == "c64" else 1e-12)
