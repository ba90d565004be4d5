"""Diagonal runs whose thread factors and constants went to another run (CPU):
circuits rich in RZ, CP and controlled RZ between dense gates, in blocks small
enough that most qubits are thread or block bits, with and without matrix-core
windows (which mix threads and end a segment), emulated op by op against the
FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_2605_15098_amd import workloads as W
from test_plan_emulator import run


@pytest.mark.parametrize("dtype,fuse,force", [(0, 0, "0"), (0, 1, "0"), (0, 5, "0"), (1, 0, "0"), (1, 1, "0"), (1, 5, "0"), (1, 5, "1")])
@pytest.mark.parametrize("n,l,logr", [(6, 3, 1), (10, 7, 2), (12, 10, 3), (13, 11, 4), (11, 11, 4)])
def test_runs_with_moved_terms(n, l, logr, dtype, fuse, force, monkeypatch):
    monkeypatch.setenv("SV_FUSE_ALL", force)
    rng = np.random.default_rng([n, l, 8])
    rows = []
    for _ in range(160):
        q, c = (int(x) for x in rng.choice(n, size=2, replace=False))
        kind = str(rng.choice(["RZ", "RZ", "P", "Z", "P", "RZ", "H", "RX", "RY", "X", "H"]))
        controlled = rng.random() < (0.5 if kind in ("RZ", "P", "Z", "X") else 0.15)
        rows.append((kind, q, c if controlled else -1, float(rng.uniform(0, 2 * np.pi))))
    g = W.gates_from_tuples(rows)
    psi0 = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi0 /= np.linalg.norm(psi0)
    got, _ = run(n, g, psi0, dtype=dtype, l=l, logr=logr, policy=2, pin=2, fuse=fuse)
    # the emulator computes in FP64; 160 gates of a few roundings each
    assert np.max(np.abs(got - oracle.apply(n, g, psi0))) < 1e-12
