"""GPU readouts in permuted layouts: export, import, probabilities, marginals
and shots through the tiled kernels against plain numpy.

A circuit of SWAP gates relabels the qubits without touching an amplitude, so
export and import have to return the imported bits, and probabilities are
sums of |a|^2 of those. Sums of at most 2^21 non-negative terms with total 1
in binary64: 1e-12 covers 2^21 roundings of 1.1e-16 with room for numpy's own.
Sizes: below, at and above a tile (2^11 amplitudes of complex64, 2^10 of
complex128), below and above the storage order's first size, 2^20 outputs.
"""
import numpy as np
import pytest

from oracle import measure as M
from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu

CD = {"c64": np.complex64, "c128": np.complex128}


def permuted(n, dtype, kind, seed):
    """A state with random amplitudes in a permuted layout, and the amplitudes in logical order."""
    rng = np.random.default_rng([seed, n])
    s = sv.StateVector(n, dtype)
    if kind == "reversed":
        pairs = [(q, n - 1 - q) for q in range(n // 2)]
    else:
        pairs = [tuple(int(x) for x in rng.choice(n, size=2, replace=False)) for _ in range(2 * n)]
    s.apply(W.gates_from_tuples([("SWAP", a, -1, 0.0, b) for a, b in pairs]))
    a = (rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)).astype(CD[dtype])
    a /= np.linalg.norm(a)
    s.set_state(a)
    assert sorted(s.layout()) == list(range(n))
    return s, a, rng


def numpy_marginal(p, n, qs):
    m = np.zeros(1 << n, dtype=np.int64)
    i = np.arange(1 << n)
    for k, q in enumerate(qs):
        m |= ((i >> q) & 1) << k
    return np.bincount(m, weights=p, minlength=1 << len(qs))


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("kind", ["reversed", "random"])
@pytest.mark.parametrize("n", [2, 9, 10, 11, 12, 15, 20])
def test_export_import(n, kind, dtype):
    import torch
    print(f"case export n={n} {kind} {dtype}", flush=True)
    s, a, rng = permuted(n, dtype, kind, 31)
    try:
        assert np.array_equal(s.state(), a)
        out = torch.zeros(1 << n, dtype=getattr(torch, "complex64" if dtype == "c64" else "complex128"), device="cuda")
        sv.sv_state(s.h, n, dtype, out=out)
        assert np.array_equal(out.cpu().numpy(), a)
        # ranges: aligned powers of two (tiles), and ones that are not
        N = 1 << n
        for off, cnt in ((0, N // 2 or 1), (N // 2, N // 2 or 1), (N // 4, N // 4 or 1), (N // 8, N // 2 or 1), (N // 3, N // 2 or 1), (N - 1, 1)):
            cnt = min(cnt, N - off)
            part = sv.sv_state_range(s.h, off, cnt, dtype, out=torch.zeros(cnt, dtype=out.dtype, device="cuda"))
            assert np.array_equal(part.cpu().numpy(), a[off:off + cnt]), (off, cnt)
            new = (rng.normal(size=cnt) + 1j * rng.normal(size=cnt)).astype(CD[dtype])
            sv.sv_set_state_range(s.h, off, torch.tensor(new, device="cuda"))
            a[off:off + cnt] = new
        assert np.array_equal(s.state(), a)
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [6, 9, 10, 13, 16, 20, 21])
def test_probabilities_and_marginals(n, dtype):
    import torch
    s, a, rng = permuted(n, dtype, "random", 32)
    try:
        p = np.abs(a.astype(np.complex128)) ** 2
        lay = s.layout()
        low = [q for q in range(n) if lay[q] < 6]    # qubits on the lanes
        subsets = [None, list(range(n)), list(range(n - 1)), list(range(1, n)), list(range(n))[::-1], low, low[:3],
                   [q for q in range(n) if q not in low], [n - 1], list(range(min(n, 8)))]
        subsets += [[int(q) for q in rng.choice(n, size=int(k), replace=False)] for k in rng.integers(1, n + 1, size=5)]
        for qs in subsets:
            if qs == [] or (qs and n - len(qs) > 12 and len(qs) > 15):
                continue
            print(f"case marginal n={n} {dtype} qubits={qs}", flush=True)
            want = p if qs is None else numpy_marginal(p, n, qs)
            out = torch.full((len(want),), -1.0, dtype=torch.float64, device="cuda")
            sv.sv_probabilities(s.h, qs, n, out=out)
            assert np.max(np.abs(out.cpu().numpy() - want)) <= 1e-12, qs
            assert np.array_equal(sv.sv_probabilities(s.h, qs, n), out.cpu().numpy()) or qs is None
    finally:
        s.close()


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n,shots", [(5, 3), (9, 4), (9, 9), (10, 15), (16, 1000), (17, 100), (20, 5000)])
@pytest.mark.parametrize("layout", ["identity", "permuted"])
def test_shots_with_and_without_table(n, shots, layout, dtype):
    """Around the M / 64 shots where the table of cumulative sums takes over; half of the outcomes impossible."""
    s, a, rng = permuted(n, dtype, "random", 33)
    try:
        if layout == "identity":
            s.reset()
        a[rng.random(1 << n) < 0.5] = 0
        a[: (1 << n) // 4] = 0           # whole tiles of impossible outcomes
        a[-1] = 0
        s.set_state(a)
        p = np.abs(a.astype(np.complex128)) ** 2
        u = rng.random(shots)
        u[0] = 0.0
        if shots > 1:
            u[1] = np.nextafter(1.0, 0.0)
        print(f"case shots n={n} shots={shots} {layout} {dtype}", flush=True)
        for qs in (None, list(range(n))[::-1]):
            got = sv.sv_sample(s.h, qs, u)
            q = p if qs is None else numpy_marginal(p, n, qs)
            want = M.sample_from(q, u)
            c, t = M.cdf(q), u * M.cdf(q)[-1]
            assert np.all(q[got.astype(np.int64)] > 0)
            for g, w, x in zip(got.tolist(), want.tolist(), t.tolist()):
                # equal, or the uniform within the sums' rounding of the CDF between the two
                assert g == w or abs(c[min(g, w)] - x) <= 1e-12 * c[-1], (g, w)
        m, pm = sv.sv_measure(s.h, None, float(u[-1]))
        assert abs(pm - p[m]) <= 1e-15 and p[m] > 0
        after = s.state()
        assert np.count_nonzero(after) == 1 and abs(abs(after[m]) - 1.0) <= 1e-6
    finally:
        s.close()
