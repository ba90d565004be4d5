"""Host code of the library over a stand-in for the HIP runtime (CPU).

tests/emu/fake_hip.cpp defines the runtime's entry points in the program that
the library is linked into, so calls on states of up to 2^36 amplitudes run here
without a GPU or their memory: what is checked is what the host side launches,
returns and keeps. The stand-in refuses a launch of 2^32 threads in one
dimension, as the runtime does.
"""
import os
import subprocess

import pytest

from paper_2605_15098_amd import sv

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
SRC = os.path.join(HERE, "emu", "fake_hip.cpp")
LIBDIR = os.path.join(ROOT, "paper_2605_15098_amd")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    """Runs the stand-in program: host(*args, **environment) -> its lines, split."""
    sv.load()  # built
    exe = str(tmp_path_factory.mktemp("host") / "fake_hip")
    subprocess.run(["g++", "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", "-o", exe, SRC, "-rdynamic",
                    os.path.join(LIBDIR, "libsvmi.so"), f"-Wl,-rpath,{LIBDIR}", f"-Wl,-rpath-link,{ROCM}/lib"], check=True)

    def run(*args, **env):
        out = subprocess.run([exe, *map(str, args)], env=dict(os.environ, SV_JIT="0", **env), check=True,
                             capture_output=True, text=True, timeout=100).stdout
        return [line.split() for line in out.splitlines()]

    return run


def calls(lines):
    """{name: (status, launches, most threads of a launch)}"""
    return {name: tuple(int(x) for x in rest) for name, *rest in lines}


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [1, 14, 30, 31, 32, 33, 34, 35, 36])
def test_reset_of_every_size(host, n, dtype):
    """A launch per 32 GiB (2^31 threads of 16 bytes), 16 GiB where a buffer starts between two 16-byte units."""
    got = calls(host("reset", n, dtype))
    nbytes = (16 if dtype else 8) << n
    for name, unit in (("create", 16), ("reset", 16), ("reset_between_units", 8)):
        status, launches, threads = got[name]
        units = nbytes // unit
        assert status == 0 and launches == max(1, units >> 31), (name, got[name])
        assert threads == max(256, min(units, 1 << 31)), (name, got[name])
    assert got["wrap"][0] == 0


@pytest.mark.parametrize("dtype", [0, 1])
@pytest.mark.parametrize("n", [20, 30, 32, 33, 34, 35, 36])
def test_no_launch_is_too_large(host, n, dtype):
    """Every call that sweeps the state, in the identity and in a permuted layout (shots are drawn of at most 32 qubits)."""
    seen = host("sweeps", n, dtype)
    assert len(seen) == 1 + 2 * 19
    for name, status, _, threads in seen:
        want = sv.SV_ERR_UNSUPPORTED if name == "sample" and n > 32 else 0
        assert int(status) == want and int(threads) <= 1 << 31, (name, status, threads)


def test_reset_that_fails_leaves_the_layout(host):
    """The amplitudes stay in the permuted layout when the launch fails; the next reset succeeds."""
    got = host("failed_reset")
    assert got[0][:2] == ["swap", "0"]
    assert got[1][:2] == ["reset", str(sv.SV_ERR_DEVICE)] and got[2] == ["layout", "3", "4", "2", "0", "1"]
    assert got[3][:2] == ["reset", "0"] and got[4] == ["layout", "0", "1", "2", "3", "4"]


def test_null_gate_array(host):
    """Refused also where a plan of that many gates is kept."""
    assert [(name, int(status)) for name, status, *_ in host("null_gates")] == \
        [("apply", 0), ("null", sv.SV_ERR_INVALID_ARG), ("apply", 0)]


def test_network_workspace_of_the_largest_batch():
    """128 rows of partial gradients from 2048 samples on, up to the largest int."""
    row = 4 * (sv.sv_mlp_param_count(1) + 1)
    for batch, rows in ((1, 1), (16, 1), (17, 2), (2048, 128), (2049, 128), ((1 << 31) - 17, 128), ((1 << 31) - 1, 128)):
        assert sv.sv_mlp_workspace_bytes(1, batch) == rows * row, batch


def test_kept_batches_are_compared_whole(host):
    """A batch replays the graph of equal inputs only: not that of gate lists with an equal hash, nor one planned
    under another fusion rule."""
    got = host("batch")
    assert all(line[1] == "0" for line in got if line[0] != "graphs")
    assert [int(line[1]) for line in got if line[0] == "graphs"] == [1, 1, 2, 3, 3]


@pytest.mark.parametrize("dtype,n", [("c128", 16), ("c128", 18), ("c128", 20), ("c128", 24), ("c64", 16), ("c64", 24)])
def test_exhaustive_tuner_times_the_default(host, dtype, n):
    """With device times that grow with the LDS of the launches, the default's smaller blocks of complex128 win;
    elsewhere the pick is a candidate, and where the default is one nothing else is timed."""
    got = host("tune", n, sv.DTYPES[dtype])
    pick, default = (tuple(int(x) for x in line[1:]) for line in got[1:])
    assert got[0][1] == "0"
    listed = {(c.block_qubits, c.reg_qubits, c.pin_qubits) for c in sv.sv_tune_candidates(n, dtype)}
    assert pick in listed | {default}
    if dtype == "c128" and n <= 18:
        assert default not in listed and pick == default


@pytest.mark.parametrize("dtype,ns,default", [("c64", (12, 22), True), ("c64", (12, 14), False), ("c64", (10, 18), True),
                                              ("c128", (12, 22), True)])
def test_batch_tuner_times_the_default(host, dtype, ns, default):
    """With device times that count launches and then their LDS, the default's pins win where they save a pass;
    where the default is planned like a candidate, the pick is a candidate."""
    got = host("tune_batch", *ns, sv.DTYPES[dtype])
    assert got[0][1] == "0" and got[2][1] == "0"
    block, reg, pin = (int(x) for x in got[1][1:])
    assert (block, reg, pin) == (0, 0, 0) if default else block >= 7 and reg >= 3


def test_failed_allocation_is_not_the_next_calls_error(host):
    """The runtime keeps a failed allocation's error until it is asked for one; the launch after it must not get it."""
    assert [(name, int(status)) for name, status, *_ in host("failed_allocation")] == \
        [("probabilities", sv.SV_ERR_OUT_OF_MEMORY), ("norm", sv.SV_ERR_OUT_OF_MEMORY), ("reset", 0), ("norm", 0)]


@pytest.mark.parametrize("dtype,n,log_shots,permuted,how", [
    # complex128 straight from the state only within the caches
    (1, 18, 11, 0, "state"), (1, 18, 12, 0, "table"), (1, 20, 0, 0, "state"), (1, 20, 11, 0, "array"), (1, 21, 11, 0, "state"),
    (1, 21, 12, 0, "array"), (1, 22, 0, 0, "array"), (1, 26, 0, 0, "array"), (1, 26, 19, 0, "array"),
    (1, 26, 20, 0, "table"), (1, 26, -1, 0, "array"),
    (0, 20, 13, 0, "state"), (0, 20, 14, 0, "table"), (0, 21, 14, 0, "state"), (0, 22, 15, 0, "state"), (0, 22, 16, 0, "table"),
    (0, 24, 16, 0, "state"), (0, 24, 17, 0, "array"), (0, 24, 18, 0, "table"), (0, 25, 18, 1, "array"), (0, 25, 19, 1, "table"),
    (0, 26, 0, 0, "state"), (0, 26, -1, 0, "state"), (0, 26, 18, 0, "state"), (0, 26, 19, 0, "array"), (0, 26, 20, 0, "table"),
    (0, 11, 0, 0, "state"), (0, 11, 0, 1, "table"), (0, 12, 0, 1, "array"), (1, 26, 0, 1, "array"), (0, 26, 20, 1, "table")])
def test_how_shots_are_drawn(host, dtype, n, log_shots, permuted, how):
    """By the scratch: tile sums (M / 64 bytes), with the probabilities (8 M more), or those and the table (16 M)."""
    got = host("shots", n, dtype, log_shots, permuted, 0)
    M, extra = 1 << n, 16 << max(log_shots, 5)
    scratch = int(got[1][1])
    # (a measurement of all zeros ends with an error, after the draw)
    assert int(got[0][1]) == (sv.SV_ERR_INVALID_ARG if log_shots < 0 else 0)
    least = {"state": 0, "array": 8 * M, "table": 16 * M}[how]
    assert least <= scratch <= least + M // 32 + extra + 4096, scratch
    if not permuted:
        # where there is no memory for the array, straight from the state
        few = host("shots", n, dtype, log_shots, permuted, 1)
        assert few[0][1] == got[0][1]


@pytest.mark.parametrize("n,nq", [(24, 19), (24, 18), (24, 15), (24, 13), (26, 16), (26, 19), (23, 19), (20, 14), (16, 11)])
def test_waves_of_a_marginal(host, n, nq):
    """Of the low qubits: a row of 64 outputs each, and no more waves than 2^13 (from 24 qubits on 2^15, from 26 on 2^16) or one a row."""
    (_, status, launches, threads), = host("marginal", n, nq, 0)
    rows, summed = 1 << (nq - 6), 1 << (n - nq)
    waves = max(1, min(16, summed, (1 << (13 if n < 24 else 15 if n < 26 else 16)) // rows))
    assert int(status) == 0 and int(launches) == 1 and int(threads) == 64 * rows * waves


@pytest.mark.parametrize("n,nq,high,threads", [(18, 18, 1, 1 << 18), (22, 19, 3, 64 << 13), (22, 18, 4, 64 << 13), (22, 17, 5, 64 << 13), (23, 18, 5, 64 << 14),
                                               (23, 20, 3, 256 << 9), (22, 20, 2, 256 << 9), (22, 19, 0, 64 << 13), (16, 15, 1, 64 << 7), (21, 20, 1, 256 << 9),
                                               (22, 21, 1, 256 << 10), (10, 8, 2, 64 << 2)])
def test_few_terms(host, n, nq, high, threads):
    """Without the `high` lowest qubits: a wave for eight rows of up to four terms or for one of more, a work-group
    per tile of 2^11 from 2^20 outputs on, and a thread per output where nothing is summed of a state below 2^20."""
    (_, status, launches, got), = host("marginal", n, nq, high)
    assert int(status) == 0 and int(launches) == 1 and int(got) == threads
