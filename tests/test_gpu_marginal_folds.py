"""Marginals whose summed qubits lie on a wave's lanes, on rows of them and both,
against plain numpy.

A wave folds eight rows together: half of the rows at each summed lane bit, then
the lane bits left. The cases have each number of lane bits summed with each
number of summed qubits outside the lanes from none to eight terms and more,
by rows (10 qubits: fewer than eight of them) and by tiles of 2^11 outputs.
Both sides add terms in some order in binary64: 2 (terms + 4) roundings of
2^-53 relative to the sum, which has no negative term.
"""
import numpy as np
import pytest

from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("layout", ["identity", "permuted"])
@pytest.mark.parametrize("n,cases", [(10, [(ls, ns) for ls in range(7) for ns in range(5)]), (14, [(ls, ns) for ls in range(7) for ns in range(5)]),
                                     (21, [(0, 0), (1, 0), (0, 1), (2, 1), (6, 0), (6, 2), (5, 3), (4, 3)]),
                                     (23, [(3, 0), (2, 1), (1, 2), (0, 3), (0, 2), (1, 1), (2, 0), (4, 0), (6, 1)])])
def test_lane_bits_summed(n, cases, layout, dtype):
    import torch
    rng = np.random.default_rng(n)
    s = sv.StateVector(n, dtype)
    try:
        if layout == "permuted":
            s.apply(W.gates_from_tuples([("SWAP", int(a), -1, 0.0, int(b)) for a, b in (rng.choice(n, 2, replace=False) for _ in range(2 * n))]))
        a = (rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)).astype(np.complex64 if dtype == "c64" else np.complex128)
        s.set_state(a / np.linalg.norm(a))
        a = s.state().astype(np.complex128)
        p = (a.real ** 2 + a.imag ** 2).reshape((2,) * n)
        bit_of = s.layout()                       # of a qubit
        lanes, others = [q for q in range(n) if bit_of[q] < 6], [q for q in range(n) if bit_of[q] >= 6]
        for ls, ns in cases:
            out_of = [int(q) for q in rng.choice(lanes, ls, replace=False)] + [int(q) for q in rng.choice(others, min(ns, len(others)), replace=False)]
            kept = [q for q in range(n) if q not in out_of]
            if not kept:
                continue
            if rng.random() < 0.5:
                rng.shuffle(kept)
            kept = [int(q) for q in kept]
            print(f"case n={n} {dtype} {layout} summed={out_of} kept={kept}", flush=True)
            # axis n - 1 - q is qubit q; the marginal's qubit k is its bit k
            want = p.sum(axis=tuple(n - 1 - q for q in out_of))
            order = sorted(kept, reverse=True)
            want = want.transpose([order.index(q) for q in reversed(kept)]).reshape(-1)
            got = torch.full((len(want),), -7.0, dtype=torch.float64, device="cuda")
            sv.sv_probabilities(s.h, kept, n, out=got)
            assert np.all(np.abs(got.cpu().numpy() - want) <= 2 * ((1 << len(out_of)) + 4) * 2.0 ** -53 * want), out_of
    finally:
        s.close()
