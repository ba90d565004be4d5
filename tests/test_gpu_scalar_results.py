"""Scalar results written to pinned host memory: norms and phase readouts of
many handles on several streams and threads at once, each call its own line,
equal to what the same calls give one after another."""
import threading

import numpy as np
import pytest
import torch

from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_scalar_results_of_many_threads(dtype):
    count, rounds = 12, 8
    rng = np.random.default_rng(5)
    states, want = [], []
    for i in range(count):
        n = 6 + i % 8
        s = sv.StateVector(n, dtype)
        s.apply(W.qpe_gates(n, float(rng.random())))
        states.append(s)
        want.append((s.qpe_readout(), s.norm()))
    torch.cuda.synchronize()
    got = [[] for _ in range(count)]

    def work(i):
        stream = torch.cuda.Stream()
        sv.sv_set_stream(states[i].h, stream.cuda_stream)
        for _ in range(rounds):
            got[i].append((states[i].qpe_readout(), states[i].norm()))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(count)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for i in range(count):
        assert got[i] == [want[i]] * rounds, i
    for s in states:
        s.close()
