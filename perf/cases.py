"""The work this simulator is measured on.

Each case is one job as a program does it: what it has in hand (a handle, the
gate list, input arrays, output buffers on the device) is made by
``prepare``; ``run`` is one job through the public calls; ``exact`` is what
the job's outputs are in 64-bit arithmetic, from closed forms or from plain
torch tensor products.

Kinds of job:
  qpe       phase estimation from |0...0>: reset, circuit, phase readout, and
            the state (or the counting register's distribution). The phase is
            the seed's, so another seed is another circuit of the same shape.
  circuit   a state computed elsewhere (a checkpoint) is imported, a circuit
            runs on it, the result is exported, all in device memory.
  batch     many phase estimations of uneven size in one launch, each
            instance's state read out.
  unitaries dense k-qubit unitaries, some of them controlled, on a resident
            state, then the export.
  measure   marginals over several qubit subsets, the norm and shots.
  mlp       training steps of the schedule cost model, then its predictions.
"""
import math

import numpy as np
import torch

from paper_2605_15098_amd import sv
from paper_2605_15098_amd import workloads as W

REAL = {"c64": torch.float32, "c128": torch.float64}
CPLX = {"c64": torch.complex64, "c128": torch.complex128}
BYTES = {"c64": 8, "c128": 16}


def listed():
    return [
        # the 10-qubit phase estimation of the plain method: the smallest job, all latency
        {"name": "qpe10-c128-plain", "kind": "qpe", "n": 10, "dtype": "c128", "mode": "plain", "out": "state"},
        # a small register with the default schedule: a few microseconds of kernels, so the host path shows
        {"name": "qpe17-c64", "kind": "qpe", "n": 17, "dtype": "c64", "mode": "default", "out": "state"},
        # an ordinary size whose state stays in the caches
        {"name": "qpe23-c64", "kind": "qpe", "n": 23, "dtype": "c64", "mode": "default", "out": "state"},
        # the 28-qubit double precision estimation, read out as the counting register's distribution
        {"name": "qpe28-c128", "kind": "qpe", "n": 28, "dtype": "c128", "mode": "default", "out": "counting"},
        # the largest: the inverse QFT (the gates of the large phase estimation) on an imported 8 GiB state, HBM bound
        {"name": "qft30-c64", "kind": "circuit", "n": 30, "dtype": "c64", "circuit": "qft", "depth": 1, "number": 0, "fuse_k": 1},
        # a 200-gate random circuit of the kinds the learned schedule is evaluated on
        {"name": "random27-c64", "kind": "circuit", "n": 27, "dtype": "c64", "circuit": "random", "depth": 200, "number": 7, "fuse_k": 1},
        # layers of rotations and CNOT ladders in double precision: dense 2x2 work
        {"name": "layered24-c128", "kind": "circuit", "n": 24, "dtype": "c128", "circuit": "layered", "depth": 3, "number": 3, "fuse_k": 1},
        # deep dense groups, where fused windows run on the matrix cores
        {"name": "blocked25-c64-fused", "kind": "circuit", "n": 25, "dtype": "c64", "circuit": "blocked", "depth": 24, "number": 24, "fuse_k": 5},
        # the batch of 256 uneven phase estimations
        {"name": "batch256-c64", "kind": "batch", "dtype": "c64", "count": 256, "lo": 12, "hi": 22, "sizes": 4},
        # k-qubit unitaries of every width, as a front end or a fusing compiler hands them over
        {"name": "unitaries26-c64", "kind": "unitaries", "n": 26, "dtype": "c64", "gates": 12, "number": 1},
        # the meters: marginals of several shapes and shots
        {"name": "measure25-c64", "kind": "measure", "n": 25, "dtype": "c64", "shots": 20000, "number": 1},
        # the cost model's training: eight minibatches and the predictions of its training set
        {"name": "mlp128", "kind": "mlp", "batch": 128, "steps": 8, "rows": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["qpe", "qpe", "circuit", "circuit", "batch", "unitaries", "measure", "mlp"])
    dtype = rng.choice(["c64", "c64", "c128"])
    if kind == "qpe":
        plain = rng.random() < 0.2
        # (the far tail of a larger estimation is below what single precision resolves)
        n = rng.randint(6, 20) if plain else rng.randint(8, 23 if dtype == "c64" else 28)
        return {"kind": kind, "n": n, "dtype": dtype, "mode": "plain" if plain else "default", "out": rng.choice(["state", "counting"])}
    if kind == "circuit":
        c = rng.choice(["random", "layered", "blocked", "qft"])
        depth = {"qft": 1, "random": rng.randint(40, 220), "layered": rng.randint(1, 4), "blocked": rng.randint(4, 24)}[c]
        fuse = 5 if c == "blocked" and rng.random() < 0.7 else 1
        top = (29 if c == "qft" else 26) - (1 if dtype == "c128" else 0)
        return {"kind": kind, "n": rng.randint(12, top), "dtype": dtype, "circuit": c, "depth": depth,
                "number": rng.randint(0, 999), "fuse_k": fuse}
    if kind == "batch":
        lo = rng.randint(8, 14)
        return {"kind": kind, "dtype": dtype, "count": _log_int(rng, 8, 200), "lo": lo, "hi": lo + rng.randint(2, 7), "sizes": rng.randint(0, 999)}
    if kind == "unitaries":
        return {"kind": kind, "n": rng.randint(13, 26 if dtype == "c64" else 25), "dtype": dtype, "gates": rng.randint(4, 14), "number": rng.randint(0, 999)}
    if kind == "measure":
        return {"kind": kind, "n": rng.randint(13, 26 if dtype == "c64" else 25), "dtype": dtype, "shots": _log_int(rng, 100, 20000), "number": rng.randint(0, 999)}
    return {"kind": "mlp", "batch": _log_int(rng, 32, 1024), "steps": rng.randint(2, 12), "rows": _log_int(rng, 24, 10000)}


# ------------------------------------------------------------------ inputs

def _phi(case, seed):
    return float(np.random.default_rng([seed, 11]).random())


def _gates(case):
    """The circuit of a "circuit" case: fixed by the case, not by the seed."""
    rng = np.random.default_rng([case["number"], 5])
    n, d = case["n"], case["depth"]
    if case["circuit"] == "qft":
        return W.qft_inverse_gates(n)
    if case["circuit"] == "random":
        return W.random_circuit(n, d, rng)
    if case["circuit"] == "layered":
        return W.layered_dense_circuit(n, d, rng)
    return W.blocked_dense_circuit(n, 2, d, rng)


def _random_state(n, dtype, seed):
    """A normalized state of Gaussian amplitudes (a typical entangled state)."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + n)
    x = torch.randn((1 << n, 2), generator=g, device="cuda", dtype=REAL[dtype])
    x *= 2.0 ** (-0.5 * (n + 1))
    return torch.view_as_complex(x)


def _sizes(case):
    rng = np.random.default_rng([case["sizes"], 4])
    return [int(rng.integers(case["lo"], case["hi"] + 1)) for _ in range(case["count"])]


def _phis(case, seed):
    return np.random.default_rng([seed, 12]).random(case["count"])


def _unitary_shapes(case):
    """(targets, controls) of each gate: every width from 1 to 6, qubits anywhere, every third gate controlled."""
    rng = np.random.default_rng([case["number"], 6])
    out = []
    for i in range(case["gates"]):
        k = 1 + (i + case["number"]) % 6
        c = int(rng.integers(1, 4)) if i % 3 == 2 else 0
        qs = [int(q) for q in rng.choice(case["n"], size=k + c, replace=False)]
        out.append((qs[:k], qs[k:]))
    return out


def _unitaries(case, seed):
    rng = np.random.default_rng([seed, 13])
    out = []
    for targets, controls in _unitary_shapes(case):
        d = 1 << len(targets)
        q, r = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
        out.append(("U", targets, controls, q * (np.diag(r) / np.abs(np.diag(r)))))
    return out


def _subsets(case):
    """One qubit, the low eight, a scattered ten, and all but the top qubits (the counting register's shape)."""
    n = case["n"]
    rng = np.random.default_rng([case["number"], 7])
    return [[int(rng.integers(0, n))], list(range(8)), [int(q) for q in rng.choice(n, size=10, replace=False)], list(range(n - 1))]


def _mlp_arrays(case, seed):
    """Parameters and moments as in the middle of a training run, features and targets of its scale (float64)."""
    rng = np.random.default_rng([seed, 14])
    d = sv.SV_FEATURES
    params = W.mlp_init_params(d, seed)
    rows = max(case["rows"], case["batch"])
    x = rng.normal(3.0, 4.0, size=(rows, d))
    y = 0.3 * rng.normal(size=rows) + np.tanh(x[:, :4].sum(axis=1) / 8.0)
    norm = np.concatenate([np.full(d, 3.0), np.full(d, 0.25)])
    m = 0.02 * rng.normal(size=len(params))
    v = 0.01 + 0.02 * rng.random(len(params))
    return params, x, y, norm, m, v


ADAM = {"lr": 1e-3, "beta1": 0.9, "beta2": 0.999, "eps": 1e-8, "step": 400}


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        f = [torch.tensor(a.astype(np.float32), device="cuda") for a in _mlp_arrays(case, seed)]
        params, x, y, norm, m, v = f
        d, b = sv.SV_FEATURES, case["batch"]
        return {"case": case, "params": params, "x": x, "y": y, "norm": norm, "m": m, "v": v, "grad": torch.empty_like(params),
                "loss": torch.zeros(1, device="cuda"), "ws": torch.zeros(sv.sv_mlp_workspace_bytes(d, b) // 4, device="cuda"),
                "pred": torch.empty(len(x), device="cuda"), "step": ADAM["step"]}
    dtype = case["dtype"]
    if kind == "batch":
        ns, phis = _sizes(case), _phis(case, seed)
        sims = [sv.StateVector(n, dtype) for n in ns]
        out = torch.empty(sum(1 << n for n in ns), dtype=CPLX[dtype], device="cuda")
        return {"case": case, "sims": sims, "gates": [W.qpe_gates(n, float(p)) for n, p in zip(ns, phis)], "out": out,
                "parts": list(torch.split(out, [1 << n for n in ns]))}
    n = case["n"]
    sim = sv.StateVector(n, dtype)
    if kind == "qpe":
        sched = sv.schedule("plain") if case["mode"] == "plain" else None
        out = torch.empty(1 << (n if case["out"] == "state" else n - 1), dtype=CPLX[dtype] if case["out"] == "state" else torch.float64, device="cuda")
        return {"case": case, "sim": sim, "gates": W.qpe_gates(n, _phi(case, seed)), "sched": sched, "out": out}
    if kind == "measure":
        state = _random_state(n, dtype, seed)
        sv.sv_set_state_range(sim.h, 0, state)
        subs = _subsets(case)
        rng = np.random.default_rng([seed, 15])
        return {"case": case, "sim": sim, "subsets": subs, "uniforms": rng.random(case["shots"]),
                "outs": [torch.empty(1 << len(q), dtype=torch.float64, device="cuda") for q in subs]}
    state = {"case": case, "sim": sim, "in": _random_state(n, dtype, seed), "out": torch.empty(1 << n, dtype=CPLX[dtype], device="cuda")}
    if kind == "unitaries":
        return dict(state, gates=_unitaries(case, seed))
    sched = None if case["fuse_k"] == 1 else sv.schedule(fuse_k=case["fuse_k"])
    return dict(state, gates=_gates(case), sched=sched)


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mlp":
        d, b, count = sv.SV_FEATURES, case["batch"], s["params"].numel()
        for i in range(case["steps"]):
            s["step"] += 1
            at = (i * b) % (len(s["x"]) - b + 1)
            sv.sv_mlp_grad(s["params"], d, s["norm"], s["x"][at:at + b], s["y"][at:at + b], b, s["grad"], s["loss"], s["ws"])
            sv.sv_mlp_adam(s["params"], s["m"], s["v"], s["grad"], count, ADAM["lr"], ADAM["beta1"], ADAM["beta2"], ADAM["eps"], s["step"])
        sv.sv_mlp_forward(s["params"], d, s["norm"], s["x"], len(s["x"]), s["pred"])
        return {"params": s["params"], "grad": s["grad"], "loss": s["loss"], "pred": s["pred"]}
    if kind == "batch":
        for sim in s["sims"]:
            sim.reset()
        sv.sv_apply_batch([sim.h for sim in s["sims"]], s["gates"])
        for sim, part in zip(s["sims"], s["parts"]):
            sv.sv_state(sim.h, sim.n, case["dtype"], out=part)
        return s["out"]
    sim = s["sim"]
    if kind == "qpe":
        sim.reset()
        sim.apply(s["gates"], s["sched"])
        if case["out"] == "state":
            sv.sv_state(sim.h, sim.n, case["dtype"], out=s["out"])
        else:
            sv.sv_probabilities(sim.h, list(range(sim.n - 1)), out=s["out"])
        m, phi, p = sim.qpe_readout()
        return {"m": m, "phi": phi, "p": p, "out": s["out"]}
    if kind == "measure":
        for q, out in zip(s["subsets"], s["outs"]):
            sv.sv_probabilities(sim.h, q, out=out)
        norm = sim.norm()
        shots = sv.sv_sample(sim.h, None, s["uniforms"])
        some = sv.sv_sample(sim.h, s["subsets"][2], s["uniforms"])
        return {"marginals": s["outs"], "norm": norm, "shots": shots.view(np.int64), "some": some.view(np.int64)}
    sv.sv_set_state_range(sim.h, 0, s["in"])
    if kind == "unitaries":
        sim.apply_ex(s["gates"])
    else:
        sim.apply(s["gates"], s["sched"])
    return sv.sv_state(sim.h, sim.n, case["dtype"], out=s["out"])


# ------------------------------------------------------------------ work

def _gate_flops(g):
    """Floating point operations per amplitude of one gate (an uncontrolled 2x2 product: 14)."""
    op, controlled = int(g["op"]), int(g["control"]) >= 0
    if op in (W.OP_SWAP, W.OP_X):
        return 0.0
    per = 4.0 if op == W.OP_H else (6.0 if op in (W.OP_RX, W.OP_RY) else (14.0 if op in (W.OP_U2, W.OP_Y) else 3.0))
    return per * (0.5 if controlled else 1.0)


def work(case):
    kind = case["kind"]
    if kind == "mlp":
        d, h = sv.SV_FEATURES, 64
        per = 2.0 * (d * h + h * h + h)
        count = sv.sv_mlp_param_count(d)
        rows = max(case["rows"], case["batch"])
        return {"bytes": 4.0 * (min(rows, case["batch"] * case["steps"]) * (d + 1) + rows * (d + 1) + 7 * count),
                "flops": per * (3 * case["steps"] * case["batch"] + rows)}
    if kind == "batch":
        ns = _sizes(case)
        return {"bytes": sum(float(BYTES[case["dtype"]] << n) for n in ns),
                "flops": sum(math.ldexp(sum(_gate_flops(g) for g in W.qpe_gates(n, 0.1)), n) for n in ns)}
    n, ab = case["n"], BYTES[case["dtype"]]
    state = float(ab << n)
    if kind == "qpe":
        out = state if case["out"] == "state" else 8.0 * (1 << (n - 1))
        return {"bytes": out, "flops": math.ldexp(sum(_gate_flops(g) for g in W.qpe_gates(n, 0.1)), n)}
    if kind == "measure":
        return {"bytes": state + sum(8.0 * (1 << len(q)) for q in _subsets(case)) + 32.0 * case["shots"], "flops": 4.0 * (1 << n)}
    if kind == "unitaries":
        return {"bytes": 2.0 * state, "flops": sum(math.ldexp(8.0 * (1 << len(t)), n - len(c)) for t, c in _unitary_shapes(case))}
    return {"bytes": 2.0 * state, "flops": math.ldexp(sum(_gate_flops(g) for g in _gates(case)), n)}


# ------------------------------------------------------------------ 64-bit results

def _qpe_amplitudes(t, phi):
    """Counting-register amplitudes of the phase estimation of phi on t qubits: the geometric sum
    2^-t sum_k e^{2 pi i k d}, d = phi - m / 2^t, with its phase and the sine ratio taken from reduced turns."""
    m = torch.arange(1 << t, dtype=torch.float64, device="cuda")
    scaled = math.ldexp(phi, t)
    whole = math.floor(scaled)
    frac = scaled - whole                    # exact
    off = torch.remainder(whole - m + 2.0 ** (t - 1), 2.0 ** t) - 2.0 ** (t - 1)  # signed distance in steps, less frac
    del m
    d = torch.ldexp(off + frac, torch.tensor(-t, device="cuda"))
    den = torch.sin(math.pi * d)
    num = math.sin(math.pi * frac) * (1.0 - 2.0 * torch.remainder(off, 2.0))
    mag = torch.where(den == 0, torch.ones_like(den), torch.ldexp(num / den, torch.tensor(-t, device="cuda")))
    del num, den
    # phase pi d (2^t - 1) = pi (off + frac) - pi d
    ang = torch.remainder(off, 2.0) + frac - d
    return torch.polar(mag.abs(), math.pi * (ang + (mag < 0)))


def _qpe_state(n, phi):
    out = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    out[1 << (n - 1):] = _qpe_amplitudes(n - 1, phi)
    return out


def _apply(x, n, u, targets, controls):
    """x (2^n amplitudes, qubit q = index bit q) after the 2^k x 2^k matrix u on targets where every control is 1, in place."""
    v = x.view((2,) * n)
    index = [slice(None)] * n
    for c in controls:
        index[n - 1 - c] = 1
    sub = v[tuple(index)]
    left = [q for q in range(n - 1, -1, -1) if q not in controls]
    axes = [left.index(q) for q in reversed(targets)]  # most significant row bit first
    rest = [a for a in range(len(left)) if a not in axes]
    k = len(targets)
    moved = sub.permute(axes + rest)
    y = (u @ moved.reshape(1 << k, -1)).view(moved.shape)
    moved.copy_(y)


def _marginal(p, n, qubits):
    """p (2^n probabilities) summed over the qubits not listed; bit k of the result's index is qubits[k]."""
    for b in range(n - 1, -1, -1):
        if b not in qubits:
            p = p.view(-1, 2, 1 << b).sum(dim=1).view(-1)
    m = torch.arange(1 << len(qubits), device="cuda")
    at = torch.zeros_like(m)
    for k, q in enumerate(qubits):
        at |= ((m >> k) & 1) << sorted(qubits).index(q)
    return p[at]


_M = {
    W.OP_H: [[math.sqrt(0.5), math.sqrt(0.5)], [math.sqrt(0.5), -math.sqrt(0.5)]],
    W.OP_X: [[0, 1], [1, 0]],
    W.OP_Z: [[1, 0], [0, -1]],
}


def _apply_gate(x, n, g):
    """One gate of a circuit, elementwise in complex128: a view of the state splits it at the target."""
    op, t, c, th = int(g["op"]), int(g["target"]), int(g["control"]), float(g["theta"])
    if c < 0:
        v = x.view(-1, 2, 1 << t)
        a, b = v[:, 0], v[:, 1]
    else:
        hi, lo = max(t, c), min(t, c)
        v = x.view(-1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
        a, b = (v[:, 1, :, 0], v[:, 1, :, 1]) if c > t else (v[:, 0, :, 1], v[:, 1, :, 1])
    ch, sh = math.cos(0.5 * th), math.sin(0.5 * th)
    if op == W.OP_P:
        b *= complex(math.cos(th), math.sin(th))
    elif op == W.OP_Z:
        b.neg_()
    elif op == W.OP_RZ:
        a *= complex(ch, -sh)
        b *= complex(ch, sh)
    else:
        u = _M[op] if op in _M else ([[ch, -1j * sh], [-1j * sh, ch]] if op == W.OP_RX else [[ch, -sh], [sh, ch]])
        na = u[0][0] * a + u[0][1] * b
        b.copy_(u[1][0] * a + u[1][1] * b)
        a.copy_(na)


def exact(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        return _mlp_exact(case, seed)
    if kind == "batch":
        return torch.cat([_qpe_state(n, float(p)) for n, p in zip(_sizes(case), _phis(case, seed))])
    n, dtype = case["n"], case["dtype"]
    if kind == "qpe":
        phi, t = _phi(case, seed), n - 1
        amp = _qpe_amplitudes(t, phi)
        prob = amp.abs().square()
        m = int(prob.argmax())
        p = float(prob[m])
        if case["out"] == "state":
            del prob
            out = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
            out[1 << t:] = amp
        else:
            out = prob
        return {"m": m, "phi": m / 2.0 ** t, "p": p, "out": out}
    x = _random_state(n, dtype, seed).to(torch.complex128)
    if kind == "measure":
        p = x.abs().square()
        return {"marginals": [_marginal(p, n, q) for q in _subsets(case)], "norm": float(p.sum()), "shots": None, "some": None}
    if kind == "unitaries":
        for _, targets, controls, u in _unitaries(case, seed):
            _apply(x, n, torch.tensor(u, device="cuda"), targets, controls)
        return x
    if case["circuit"] == "qft":
        return torch.fft.fft(x, norm="ortho")
    for g in _gates(case):
        _apply_gate(x, n, g)
    return x


def _mlp_exact(case, seed):
    params, x, y, norm, m, v = (torch.tensor(a.astype(np.float32).astype(np.float64), device="cuda") for a in _mlp_arrays(case, seed))
    d, h, b = sv.SV_FEATURES, 64, case["batch"]
    cut = np.cumsum([h * d, h, h * h, h, h]).tolist()

    def forward(rows):
        w1, b1, w2, b2, w3, b3 = torch.tensor_split(params, cut)
        z = (rows - norm[:d]) * norm[d:]
        h1 = torch.relu(z @ w1.view(h, d).t() + b1)
        h2 = torch.relu(h1 @ w2.view(h, h).t() + b2)
        return z, h1, h2, h2 @ w3 + b3

    step, grad, loss = ADAM["step"], None, None
    for i in range(case["steps"]):
        step += 1
        at = (i * b) % (len(x) - b + 1)
        z, h1, h2, out = forward(x[at:at + b])
        r = out - y[at:at + b]
        loss = (r * r).mean()
        _, _, w2, _, w3, _ = torch.tensor_split(params, cut)
        dy = 2.0 * r / b
        g2 = dy[:, None] * w3 * (h2 > 0)
        g1 = (g2 @ w2.view(h, h)) * (h1 > 0)
        grad = torch.cat([(g1.t() @ z).reshape(-1), g1.sum(0), (g2.t() @ h1).reshape(-1), g2.sum(0), h2.t() @ dy, dy.sum().view(1)])
        m = ADAM["beta1"] * m + (1 - ADAM["beta1"]) * grad
        v = ADAM["beta2"] * v + (1 - ADAM["beta2"]) * grad * grad
        mh, vh = m / (1 - ADAM["beta1"] ** step), v / (1 - ADAM["beta2"] ** step)
        params = params - ADAM["lr"] * mh / (vh.sqrt() + ADAM["eps"])
    return {"params": params, "grad": grad, "loss": loss.view(1), "pred": forward(x)[3]}
