"""Workloads of the library's public entry points over the sizes its users run.

listed() names twelve fixed workloads, draw() makes one more of the same ranges, prepare() builds
what a program holds before the call (circuit, noise strengths, buffers, handles), run() is one
pass through the public calls, work() the bytes and operations one pass cannot do without, and
exact() the same outputs from plain 64-bit torch and numpy.

The kinds:
  traj      run_trajectories: the ideal circuit and T noisy trajectories (the paper's Monte Carlo
            method), with the fused plan the library picks.
  graph     the same through a captured TrajGraph: many short passes, launch-bound.
  dm        dm_run: the exact density matrix of a noisy circuit through the fused passes.
  channels  the density matrix one call at a time: dm_apply_gate, apply_kraus, dm_fidelity (how
            relative states under T1 / T2 relaxation are computed).
  fixed     the fixed-rank density matrix, apply_noisy_gate step by step.
  gates     a state vector one gate at a time: apply_gate, then fidelity.

Every gate of `fixed` has a strength of its own, as the gates of a calibrated device do; with one
strength for all gates eigenvalues tie and the kept eigenvectors are arbitrary inside a tie.

complex<float> runs promise single precision (their fidelities within 1e-5), so their scalar
results are handed on as float32; complex<double> runs hand on float64.
"""
import math
from dataclasses import dataclass
from typing import Optional

import numpy as np
import torch

import paper_1412_2293_amd as q

# gate kinds and noise tags of the C interface
U1, CP, SWAP, CNOT, U2, FLIP = 0, 1, 2, 3, 4, 5
ROT, PHASE = 1, 2
HADAMARD = np.array([[1.0, 1.0], [1.0, -1.0]], np.complex128) / math.sqrt(2.0)


# ------------------------------------------------------------------------------------------
# The cases
# ------------------------------------------------------------------------------------------
def listed():
    return [
        # the plain method's configuration: 200 trajectories of Grover on 10 qubits, the whole
        # circuit (25 iterations) on states that fit one tile -- the smallest trajectory call
        {"name": "traj_grover10", "kind": "traj", "circuit": "grover", "n": 10, "layers": 25, "T": 200, "dtype": "c128"},
        # the headline circuit: QFT on 26 qubits from a basis state, noisy Hadamards and phases
        {"name": "traj_qft26", "kind": "traj", "circuit": "qft", "n": 26, "layers": 1, "T": 16, "dtype": "c64"},
        # a request of the serving stream: random layers with random pairs, mid-size, odd T
        {"name": "traj_random22", "kind": "traj", "circuit": "random", "n": 22, "layers": 4, "T": 40, "dtype": "c64"},
        # large states in double precision: brickwork random layers on 26 qubits
        {"name": "traj_brick26", "kind": "traj", "circuit": "brickwork", "n": 26, "layers": 3, "T": 6, "dtype": "c128"},
        # Grover at a size bound by HBM: the first iterations of the 20-qubit search
        {"name": "traj_grover20", "kind": "traj", "circuit": "grover", "n": 20, "layers": 16, "T": 64, "dtype": "c64"},
        # launch-bound replay: random pairs on 14 qubits, 60 layers, 16 trajectories
        {"name": "graph_random14", "kind": "graph", "circuit": "random", "n": 14, "layers": 60, "T": 16, "dtype": "c64"},
        # exact density matrix of Grover on 13 qubits (2^26 entries), eight iterations
        {"name": "dm_grover13", "kind": "dm", "circuit": "grover", "n": 13, "layers": 8, "T": 1, "dtype": "c128"},
        # exact density matrix of the QFT: noisy Hadamards and averaged noisy phases
        {"name": "dm_qft12", "kind": "dm", "circuit": "qft", "n": 12, "layers": 1, "T": 1, "dtype": "c64"},
        # channels one call at a time on 11 qubits: gates, relaxation, two-qubit Kraus pairs
        {"name": "channels11", "kind": "channels", "circuit": "relax", "n": 11, "layers": 1, "T": 1, "dtype": "c128"},
        # fixed rank at its full-size configuration: Grover on 24 qubits, rank 8, first iteration
        {"name": "fixed_grover24", "kind": "fixed", "circuit": "grover", "n": 24, "layers": 1, "T": 1, "dtype": "c64"},
        # fixed rank with two-qubit Kraus steps: QFT on 17 qubits with noisy phases, rank 8
        {"name": "fixed_qft17", "kind": "fixed", "circuit": "qft", "n": 17, "layers": 1, "T": 1, "dtype": "c128"},
        # a large state gate by gate: every gate kind on low, middle and high qubits
        {"name": "gates27", "kind": "gates", "circuit": "sweeps", "n": 27, "layers": 1, "T": 1, "dtype": "c64"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed ranges: no larger in state bytes, and no more work, than the largest
    listed case of its kind."""
    kind = rng.choice(["traj", "traj", "traj", "graph", "dm", "channels", "fixed", "gates"])
    dtype = rng.choice(["c64", "c128"])
    amp = 8 if dtype == "c64" else 16
    c = {"kind": kind, "dtype": dtype}
    if kind == "traj":
        c["circuit"] = rng.choice(["grover", "qft", "random", "brickwork"])
        c["n"] = rng.randint(8, 26)
        room = (1 << 33) // (amp << c["n"])               # slots in 8 GiB
        c["T"] = _log_int(rng, 1, min(200, room - 1))
        c["layers"] = 1 if c["circuit"] == "qft" else _log_int(rng, 1, 25)
        while c["layers"] > 1 and work(c)["flops"] > 5e11:
            c["layers"] //= 2
        while c["T"] > 1 and work(c)["flops"] > 5e11:
            c["T"] //= 2
    elif kind == "graph":
        c["circuit"] = rng.choice(["random", "grover"])
        c["n"], c["T"], c["layers"] = rng.randint(11, 16), _log_int(rng, 2, 24), rng.randint(4, 30)
    elif kind == "dm":
        c["circuit"] = rng.choice(["grover", "qft"])
        c["n"], c["T"] = rng.randint(6, 13), 1
        c["layers"] = rng.randint(1, 8) if c["circuit"] == "grover" else 1
    elif kind == "channels":
        c["circuit"], c["n"], c["T"], c["layers"] = "relax", rng.randint(4, 11), 1, 1
    elif kind == "fixed":
        c["circuit"] = rng.choice(["grover", "qft"])
        c["n"] = rng.randint(10, 23) if c["circuit"] == "grover" else rng.randint(8, 16)
        c["T"], c["layers"] = 1, 1
    else:
        c["circuit"], c["n"], c["T"], c["layers"] = "sweeps", rng.randint(12, 27 if dtype == "c64" else 26), 1, 1
    return c


# ------------------------------------------------------------------------------------------
# Circuits (the conventions of include/qsim.h; qubit q is bit q of the amplitude index)
# ------------------------------------------------------------------------------------------
@dataclass
class Gate:
    kind: int
    q0: int = 0
    q1: int = 0
    m: Optional[np.ndarray] = None
    theta: float = 0.0
    noise: int = 0
    site: int = 0
    mask: int = 0
    value: int = 0
    e: float = 0.0            # this gate's own strength (fixed rank, channels)
    ops: Optional[np.ndarray] = None   # a Kraus set instead of a gate (channels)


def _haar(rng, dim):
    z = rng.standard_normal((dim, dim)) + 1j * rng.standard_normal((dim, dim))
    u, r = np.linalg.qr(z)
    d = np.diag(r)
    return u * (d / np.abs(d))[None, :]


def _relaxation(t, T1, T2):
    """Amplitude damping over t (T1) followed by dephasing (T2), as one Kraus set."""
    g, p = 1.0 - math.exp(-t / T1), 0.5 * (1.0 - math.exp(-t / T2))
    damp = [np.array([[1, 0], [0, math.sqrt(1 - g)]]), np.array([[0, math.sqrt(g)], [0, 0]])]
    deph = [math.sqrt(1 - p) * np.eye(2), math.sqrt(p) * np.diag([1.0, -1.0])]
    return np.array([b @ a for b in deph for a in damp], np.complex128)


def _cp_pair(theta, e):
    """Kraus pair of a noisy controlled phase in its improved form (eq. 14)."""
    P = math.exp(-e * e)
    f = (math.sqrt(1 + 3 * P) - 1 - P) / math.sqrt(P * (1 - P))
    k = 1.0 / math.sqrt(1 + f * f)
    u = np.exp(-1j * theta)
    return np.array([np.diag([k, k, k, u * k * (math.sqrt(P) + f * math.sqrt(1 - P))]),
                     np.diag([-f * k, -f * k, -f * k, u * k * (math.sqrt(1 - P) - f * math.sqrt(P))])], np.complex128)


def _circuit(case, seed):
    """(gates, initial index, marked index or -1)."""
    n, layers = case["n"], case["layers"]
    rng = np.random.default_rng([seed, n, layers])
    N, full = 1 << n, (1 << n) - 1
    gates, init, marked = [], 0, -1
    kind = case["circuit"]
    if kind == "grover":
        marked = int(rng.integers(0, N))
        hs = lambda: [Gate(U1, q0=a, m=HADAMARD, noise=ROT) for a in range(n)]  # noqa: E731
        gates += hs()
        for _ in range(layers):
            gates += [Gate(FLIP, mask=full, value=marked)] + hs() + [Gate(FLIP, mask=full, value=0)] + hs()
    elif kind == "qft":
        init = int(rng.integers(0, N))
        for t in range(n - 1, -1, -1):
            gates.append(Gate(U1, q0=t, m=HADAMARD, noise=ROT))
            for c in range(t - 1, -1, -1):
                gates.append(Gate(CP, q0=c, q1=t, theta=2.0 * math.pi / (1 << (t - c + 1)), noise=PHASE))
        gates += [Gate(SWAP, q0=a, q1=n - 1 - a) for a in range(n // 2)]
    elif kind in ("random", "brickwork"):
        for layer in range(layers):
            gates += [Gate(U1, q0=a, m=_haar(rng, 2), noise=ROT) for a in range(n)]
            if kind == "random":
                p = rng.permutation(n)
                pairs = [(int(p[2 * i]), int(p[2 * i + 1])) for i in range(n // 2)]
            else:
                pairs = [(a, a + 1) for a in range(layer % 2, n - 1, 2)]
            gates += [Gate(CP, q0=min(a, b), q1=max(a, b), theta=math.pi, noise=PHASE) for a, b in pairs]
    elif kind == "relax":
        for _ in range(layers):
            for a in range(n):
                gates.append(Gate(U1, q0=a, m=_haar(rng, 2), noise=ROT, e=float(rng.uniform(0.01, 0.05))))
                gates.append(Gate(U1, q0=a, ops=_relaxation(1.0, float(rng.uniform(50, 500)), float(rng.uniform(20, 300)))))
            for a in range(0, n - 1, 2):
                b = int(rng.integers(a + 1, n))
                theta, e = float(rng.uniform(0, 2 * math.pi)), float(rng.uniform(0.01, 0.05))
                gates.append(Gate(CP, q0=a, q1=b, theta=theta, noise=PHASE, e=e))
                gates.append(Gate(CP, q0=a, q1=b, ops=_cp_pair(theta, e)))
                gates.append(Gate(CNOT, q0=b, q1=a))
    else:
        # every gate kind on low, middle and high qubits
        mid, top = n // 2, n - 1
        u = lambda a: Gate(U1, q0=a, m=_haar(rng, 2), noise=ROT, e=0.01)  # noqa: E731
        cp = lambda a, b: Gate(CP, q0=a, q1=b, theta=float(rng.uniform(0, 6)), noise=PHASE, e=0.01)  # noqa: E731
        w = lambda a, b: Gate(U2, q0=a, q1=b, m=_haar(rng, 4))  # noqa: E731
        gates = [u(0), u(4), u(mid), u(top), cp(3, top - 3), cp(mid, top), Gate(SWAP, q0=2, q1=top - 1),
                 Gate(SWAP, q0=mid, q1=top), Gate(CNOT, q0=mid, q1=top), Gate(CNOT, q0=top, q1=1), w(3, mid),
                 w(top, top - 1), w(0, 1), Gate(FLIP, mask=full, value=int(rng.integers(0, N)))]
    for i, g in enumerate(gates):
        g.site = i
    if case["kind"] == "fixed":
        # one strength per qubit: distinct, in a seeded order; a controlled phase takes its control's
        s = 0.025 * 1.03 ** rng.permutation(n)
        for g in gates:
            g.e = float(s[g.q0])
    return gates, init, marked


def _strengths(case, seed):
    """One noise strength per trajectory (0.001 ... 0.05, half of the runs one for all)."""
    rng = np.random.default_rng([seed, 7])
    if rng.random() < 0.5:
        return float(rng.uniform(0.001, 0.05))
    return rng.uniform(0.001, 0.05, case["T"])


def _random_state(n, dtype, seed, device):
    """A normalised state of complex Gaussian amplitudes."""
    g = torch.Generator(device=device).manual_seed(seed + 1)
    x = torch.randn((1 << n, 2), generator=g, device=device, dtype=torch.float32)
    x = torch.view_as_complex(x)
    x /= math.sqrt(2.0 * (1 << n))
    return x.to(torch.complex64 if dtype == "c64" else torch.complex128)


# ------------------------------------------------------------------------------------------
def prepare(case, seed):
    n, T, kind = case["n"], case["T"], case["kind"]
    dt = q.C64 if case["dtype"] == "c64" else q.C128
    gates, init, marked = _circuit(case, seed)
    s = {"kind": kind, "n": n, "T": T, "dt": dt, "init": init, "marked": marked, "seed": seed}
    if kind in ("traj", "graph"):
        s["e"] = _strengths(case, seed)
        s["ga"] = q.gate_array(gates)
        if kind == "traj":
            s["buf"] = torch.empty(q.traj_bytes_required(s["ga"], n, dt, T), dtype=torch.uint8, device="cuda")
        else:
            s["graph"] = q.TrajGraph(s["ga"], n, dt, T)
    elif kind == "dm":
        s["e"] = float(np.random.default_rng([seed, 7]).uniform(0.005, 0.05))
        s["ga"] = q.gate_array(gates)
        s["psi"] = q.StateVector(n, dt, 1)
        s["psi"].init_basis(init)
        for g in s["ga"]:
            q.apply_gate(s["psi"], g)
        s["buf"] = torch.empty(q.dm_run_bytes_required(s["ga"], n, dt, s["e"]), dtype=torch.uint8, device="cuda")
    elif kind == "channels":
        s["steps"] = [(g, None) if g.ops is not None else (g, q.gate_array([g])[0]) for g in gates]
        s["rho"] = q.StateVector(2 * n, dt, 1)
        s["psi"] = q.StateVector(n, dt, 1)
        s["psi"].amplitudes()[0].copy_(_random_state(n, case["dtype"], seed, "cuda"))
    elif kind == "fixed":
        s["gates"] = [(x, g.e) for x, g in zip(q.gate_array(gates), gates)]
        s["fr"] = q.FixedRank(n, 8, dt)
        s["psi"] = q.StateVector(n, dt, 1)
        s["psi"].init_basis(init)
        for x, _ in s["gates"]:
            q.apply_gate(s["psi"], x)
    else:
        s["gates"] = [(x, g.e) for x, g in zip(q.gate_array(gates), gates)]
        s["psi"] = q.StateVector(n, dt, 1)
        s["psi"].amplitudes()[0].copy_(_random_state(n, case["dtype"], seed, "cuda"))
        s["ref"] = q.StateVector(n, dt, 1)
        s["ref"].amplitudes()[0].copy_(_random_state(n, case["dtype"], seed + 1, "cuda"))
    return s


def _scalars(dt, *values):
    """Scalar results in the run's own precision."""
    return np.array(values, np.float32 if dt == q.C64 else np.float64)


def run(s):
    kind, n, dt = s["kind"], s["n"], s["dt"]
    if kind in ("traj", "graph"):
        if kind == "traj":
            r = q.run_trajectories(s["ga"], n, s["init"], dt, s["T"], e=s["e"], seed=s["seed"], marked=s["marked"],
                                   buf=s["buf"])
        else:
            r = s["graph"].launch(s["init"], e=s["e"], seed=s["seed"], marked=s["marked"])
        real = np.float32 if dt == q.C64 else np.float64
        out = {"F": r["F"].astype(real), "norm": r["norm"].astype(real), "layout": r["layout"],
               "states": q.trajectory_states(r, n, dt, s["T"])}
        if r["p"] is not None:
            out["p"] = r["p"].astype(real)
        return out
    if kind == "dm":
        r = q.dm_run(s["ga"], n, s["init"], dt, s["psi"], e=s["e"], buf=s["buf"])
        return {"F": _scalars(dt, r["F"], r["trace"]), "layout": r["layout"], "rho": q.dm_state(r, n, dt)}
    if kind == "channels":
        rho = s["rho"]
        rho.init_basis(0)
        for g, x in s["steps"]:
            if x is None:
                q.apply_kraus(rho, [g.q0] if g.ops.shape[1] == 2 else [g.q0, g.q1], g.ops)
            else:
                q.dm_apply_gate(rho, x, g.e)
        return {"F": _scalars(dt, *q.dm_fidelity(rho, s["psi"])), "rho": rho.amplitudes()}
    if kind == "fixed":
        fr = s["fr"]
        fr.init_basis(s["init"])
        zero_tol = 1e-13 if dt == q.C128 else 1e-6
        ranks = [fr.apply_noisy_gate(x, e, zero_tol=zero_tol) for x, e in s["gates"]]
        f = fr.fidelity(s["psi"])
        return {"F": _scalars(dt, *f), "ranks": np.array(ranks), "columns": fr.columns()[:ranks[-1]]}
    psi = s["psi"]
    for x, e in s["gates"]:
        q.apply_gate(psi, x, e, seed=s["seed"])
    f, ov = q.fidelity(psi, 0, s["ref"], 0)
    return {"F": _scalars(dt, f, ov.real, ov.imag), "psi": psi.amplitudes()}


# ------------------------------------------------------------------------------------------
def _updates(g, amps):
    """(amplitudes rewritten, operations) of one gate over `amps` amplitudes."""
    if g.ops is not None:
        d = 4 if g.ops.shape[1] == 2 else 16     # the superoperator's dimension on vec(rho)
        return amps, amps * (8 * d - 2)
    if g.kind == U1:
        return amps, amps * (6 if not np.any(np.imag(g.m)) else 14)
    if g.kind == U2:
        return amps, amps * 30
    if g.kind == CP:
        return amps // 4, amps // 4 * 6
    if g.kind in (SWAP, CNOT):
        return amps // 2, 0
    k = amps >> bin(g.mask).count("1")
    return k, 2 * k


def work(case):
    n, T, kind = case["n"], case["T"], case["kind"]
    amp = 8 if case["dtype"] == "c64" else 16
    gates, _, _ = _circuit(case, 1)
    if kind in ("traj", "graph"):
        amps = (T + 1) << n                      # every final state written once
        return {"bytes": amps * amp + 352 * len(gates), "flops": sum(_updates(g, amps)[1] for g in gates)}
    if kind == "dm":
        # every entry of rho written once; a channel or a gate on rows and columns: twice a gate's
        amps = 1 << (2 * n)
        return {"bytes": amps * amp, "flops": sum(2 * _updates(g, amps)[1] for g in gates)}
    if kind == "channels":
        # each call reads and writes the entries it changes (a gate's rows, then its columns)
        amps, b, f = 1 << (2 * n), 0, 0
        for g in gates:
            upd, ops = _updates(g, amps)
            noisy = g.ops is not None or (g.kind == U1 and g.noise)
            b += 2 * upd * amp * (1 if noisy else 2)
            f += ops * (1 if g.ops is not None else 2)
        return {"bytes": b + 2 * amps * amp, "flops": f}
    if kind == "fixed":
        # a Kraus step reads and writes the eight columns; its Gram matrix and recombination
        amps, b, f = 8 << n, 0, 0
        for g in gates:
            upd, ops = _updates(g, amps)
            if g.noise:
                k = 2 if g.kind == U1 else 4
                b += 2 * amps * amp
                f += amps * 8 * 8 * k * 3 // 2
            else:
                b += 2 * upd * amp
                f += ops
        return {"bytes": b, "flops": f}
    amps = 1 << n
    return {"bytes": sum(2 * _updates(g, amps)[0] * amp for g in gates) + 2 * amps * amp,
            "flops": sum(_updates(g, amps)[1] for g in gates) + 16 * amps}


# ------------------------------------------------------------------------------------------
# The same outputs in 64 bits (plain torch and numpy)
# ------------------------------------------------------------------------------------------
def _xi(seed, sites, T):
    """xi[t, site]: Philox4x32-10 (key seed, counter (site, t, 0, 0)), Box-Muller cosine branch."""
    M = np.uint64(0xFFFFFFFF)
    site, t = np.meshgrid(np.asarray(sites, np.uint64), np.arange(T, dtype=np.uint64))
    c = [site, t, np.zeros_like(site), np.zeros_like(site)]
    k0, k1 = np.uint64(seed & 0xFFFFFFFF), np.uint64(seed >> 32)
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
        c = [(b >> np.uint64(32)) ^ c[1] ^ k0, b & M, (a >> np.uint64(32)) ^ c[3] ^ k1, a & M]
        k0, k1 = (k0 + np.uint64(0x9E3779B9)) & M, (k1 + np.uint64(0xBB67AE85)) & M
    u1 = (((c[0] << np.uint64(32)) | c[1]) >> np.uint64(11)).astype(np.float64)
    u2 = (((c[2] << np.uint64(32)) | c[3]) >> np.uint64(11)).astype(np.float64)
    return np.sqrt(-2.0 * np.log((u1 + 1.0) * 2.0 ** -53)) * np.cos(2.0 * math.pi * (u2 * 2.0 ** -53))


def _halves(psi, bit):
    v = psi.view(psi.shape[0], -1, 2, 1 << bit)
    return v[:, :, 0], v[:, :, 1]


def _apply1(psi, bit, m):
    """m: [S or 1, 2, 2] on index bit `bit` of psi [S, N], in place."""
    x0, x1 = _halves(psi, bit)
    m = m[:, :, :, None, None]
    y0 = m[:, 0, 0] * x0 + m[:, 0, 1] * x1
    y1 = m[:, 1, 0] * x0 + m[:, 1, 1] * x1
    x0.copy_(y0)
    x1.copy_(y1)


def _quarters(psi, b0, b1):
    """Views of psi [S, N] with (bit b0, bit b1) = local index 0..3 (b0 the low local bit)."""
    lo, hi = min(b0, b1), max(b0, b1)
    v = psi.view(psi.shape[0], -1, 2, 1 << (hi - lo - 1), 2, 1 << lo)
    pick = lambda x0, x1: v[:, :, x1, :, x0] if b0 == lo else v[:, :, x0, :, x1]  # noqa: E731
    return [pick(l & 1, l >> 1) for l in range(4)]


def _apply2(psi, b0, b1, m):
    x = _quarters(psi, b0, b1)
    y = []
    for r in range(4):
        acc = None
        for c in range(4):
            if m[r, c] != 0:
                t = x[c] * complex(m[r, c])
                acc = t if acc is None else acc.add_(t)
        y.append(torch.zeros_like(x[0]) if acc is None else acc)
    for r in range(4):
        x[r].copy_(y[r])


def _pattern(psi, mask, value, factor):
    N = psi.shape[1]
    bits = N.bit_length() - 1
    free = [b for b in range(bits) if not (mask >> b) & 1]
    idx = torch.zeros(1, dtype=torch.int64, device=psi.device) + value
    for b in free:
        idx = torch.cat([idx, idx + (1 << b)])
    psi[:, idx] = psi[:, idx] * factor


_CNOT = np.array([[1, 0, 0, 0], [0, 0, 0, 1], [0, 0, 1, 0], [0, 1, 0, 0]], np.complex128)


def _noisy_u(m, a):
    """m V(a), V = [[cos, sin], [-sin, cos]], for an array of angles: [len(a), 2, 2]."""
    c, s = np.cos(a), np.sin(a)
    v = np.empty((len(a), 2, 2))
    v[:, 0, 0], v[:, 0, 1], v[:, 1, 0], v[:, 1, 1] = c, s, -s, c
    return np.asarray(m)[None] @ v


def _evolve(psi, gates, perm, ang):
    """Gates on psi [S, N]; ang(gate): per-slot angle e xi (or None).  SWAPs only relabel perm."""
    dev = psi.device
    for g in gates:
        if g.kind == SWAP:
            perm[g.q0], perm[g.q1] = perm[g.q1], perm[g.q0]
            continue
        a = ang(g)
        if g.kind == U1:
            m = _noisy_u(g.m, a) if a is not None else np.asarray(g.m)[None]
            _apply1(psi, perm[g.q0], torch.as_tensor(m, dtype=torch.complex128, device=dev))
        elif g.kind == CP:
            th = g.theta + (a if a is not None else np.zeros(1))
            w = torch.as_tensor(np.exp(-1j * th), device=dev)
            x = _quarters(psi, perm[g.q0], perm[g.q1])[3]
            x.mul_(w.view(-1, 1, 1, 1))
        elif g.kind in (CNOT, U2):
            _apply2(psi, perm[g.q0], perm[g.q1], _CNOT if g.kind == CNOT else g.m)
        else:
            mask = sum(1 << perm[b] for b in range(len(perm)) if (g.mask >> b) & 1)
            value = sum(1 << perm[b] for b in range(len(perm)) if (g.value >> b) & 1)
            _pattern(psi, mask, value, -1.0)


def _exact_traj(case, seed, dev):
    n, T = case["n"], case["T"]
    gates, init, marked = _circuit(case, seed)
    e = np.broadcast_to(np.asarray(_strengths(case, seed), np.float64), (T,))
    a = np.zeros((T + 1, len(gates)))
    a[1:] = _xi(seed, [g.site for g in gates], T) * e[:, None]
    out = torch.empty((T + 1, 1 << n), dtype=torch.complex128, device=dev)
    step = max(1, (1 << 27) >> n)
    for s0 in range(0, T + 1, step):
        psi = out[s0:s0 + step]
        psi.zero_()
        psi[:, init] = 1.0
        perm = list(range(n))
        _evolve(psi, gates, perm, lambda g: a[s0:s0 + step, g.site] if g.noise else None)
    ov = np.array([complex(torch.vdot(out[0], out[t])) for t in range(T + 1)])
    nr = np.array([float(torch.linalg.vector_norm(out[t])) ** 2 for t in range(T + 1)])
    r = {"F": np.abs(ov[1:]) ** 2 / (nr[0] * nr[1:]), "norm": nr[1:], "layout": None, "states": out}
    if marked >= 0:
        at = sum(1 << perm[b] for b in range(n) if (marked >> b) & 1)
        r["p"] = (out[1:, at].abs() ** 2).cpu().numpy()
    return r


def _superop(ops):
    """sum_k E_k (x) conj(E_k) on local index (column bits low, row bits high)."""
    return sum(np.kron(E, E.conj()) for E in ops)


def _rot_ops(m, e):
    l1, l2 = 0.5 * (1 + math.exp(-2 * e * e)), 0.5 * (1 - math.exp(-2 * e * e))
    return [m * math.sqrt(l1), math.sqrt(l2) * (m @ np.array([[0.0, 1.0], [-1.0, 0.0]]))]


def _evolve_rho(rho, n, gates, strength):
    """Channels on vec(rho) [1, 4^n], entry rho_ij at i 2^n + j; returns the relabelling."""
    perm = list(range(n))
    for g in gates:
        e = strength(g)
        if g.ops is not None and g.ops.shape[1] == 2:
            _apply2(rho, perm[g.q0], perm[g.q0] + n, _superop(g.ops))
        elif g.ops is not None:
            # two-qubit set, diagonal operators: entry (i, j) times sum_k E_k[a, a] conj(E_k[b, b])
            d = np.array([np.diag(E) for E in g.ops])
            w = torch.as_tensor(d.T @ d.conj(), device=rho.device)
            idx = torch.arange(1 << n, device=rho.device)
            loc = ((idx >> perm[g.q0]) & 1) + 2 * ((idx >> perm[g.q1]) & 1)
            rho.view(1 << n, 1 << n).mul_(w[loc][:, loc])
        elif g.kind == U1 and g.noise and e > 0:
            _apply2(rho, perm[g.q0], perm[g.q0] + n, _superop(_rot_ops(np.asarray(g.m), e)))
        elif g.kind == CP and g.noise and e > 0:
            idx = torch.arange(1 << n, device=rho.device)
            b = ((idx >> perm[g.q0]) & (idx >> perm[g.q1]) & 1).to(torch.float64)
            f = math.exp(-0.5 * e * e) * np.exp(-1j * g.theta)
            one = torch.ones((), dtype=torch.complex128, device=rho.device)
            row, col = torch.where(b > 0, one * f, one), torch.where(b > 0, one * np.conj(f), one)
            v = rho.view(1 << n, 1 << n)
            v.mul_(row[:, None]).mul_(col[None, :])
            if e > 0:
                both = (b[:, None] * b[None, :]) > 0
                v[both] *= math.exp(e * e)
        elif g.kind == SWAP:
            perm[g.q0], perm[g.q1] = perm[g.q1], perm[g.q0]
        else:
            # U on the rows, conj(U) on the columns
            for shift, conj in ((n, False), (0, True)):
                h = Gate(g.kind, g.q0, g.q1, None if g.m is None else (np.conj(g.m) if conj else g.m),
                         -g.theta if conj else g.theta, mask=g.mask, value=g.value)
                p = [x + shift for x in perm]
                if g.kind == FLIP:
                    mask = sum(1 << p[b] for b in range(n) if (g.mask >> b) & 1)
                    value = sum(1 << p[b] for b in range(n) if (g.value >> b) & 1)
                    v = rho.view(1 << n, 1 << n)
                    i = value >> shift
                    if mask >> shift == (1 << n) - 1:
                        (v[i] if shift else v[:, i]).mul_(-1.0)
                    else:
                        _pattern(rho, mask, value, -1.0)
                else:
                    _evolve(rho, [h], p, lambda _: None)
    return perm


def _exact_dm(case, seed, dev):
    n = case["n"]
    gates, init, _ = _circuit(case, seed)
    rho = torch.zeros((1, 1 << (2 * n)), dtype=torch.complex128, device=dev)
    psi = torch.zeros((1, 1 << n), dtype=torch.complex128, device=dev)
    if case["kind"] == "dm":
        rho[0, (init << n) | init] = 1.0
        psi[0, init] = 1.0
        e = float(np.random.default_rng([seed, 7]).uniform(0.005, 0.05))
        perm = list(range(n))
        _evolve(psi, gates, perm, lambda _: None)
        assert perm == _evolve_rho(rho, n, gates, lambda g: e if g.noise else 0.0)
    else:
        rho[0, 0] = 1.0
        psi[0] = _random_state(n, case["dtype"], seed, dev).to(torch.complex128)
        _evolve_rho(rho, n, gates, lambda g: g.e)
    v = rho.view(1 << n, 1 << n)
    f = complex(torch.vdot(psi[0], torch.mv(v, psi[0]))).real
    F = np.array([f, complex(torch.diagonal(v).sum()).real])
    if case["kind"] == "dm":
        return {"F": F, "layout": None, "rho": rho[0]}
    return {"F": F, "rho": rho}


def _exact_fixed(case, seed, dev):
    """The fixed-rank step in 64 bits; the columns are free up to a phase each, so only the
    fidelities and the lost weight have values."""
    n, r = case["n"], 8
    zero_tol = 1e-13 if case["dtype"] == "c128" else 1e-6
    gates, init, _ = _circuit(case, seed)
    V = torch.zeros((1, 1 << n), dtype=torch.complex128, device=dev)
    V[0, init] = 1.0
    psi = V.clone()
    perm, unused = list(range(n)), list(range(n))
    _evolve(psi, gates, unused, lambda _: None)
    log_trace = 0.0
    for g in gates:
        if not g.noise:
            if g.kind == SWAP:
                x = _quarters(V, g.q0, g.q1)
                t = x[1].clone()
                x[1].copy_(x[2])
                x[2].copy_(t)
            else:
                _evolve(V, [g], perm, lambda _: None)
            continue
        parts = []
        P = math.exp(-g.e * g.e)
        for k in range(2):
            W = V.clone()
            if g.kind == U1:
                _apply1(W, g.q0, torch.as_tensor(_rot_ops(np.asarray(g.m), g.e)[k][None], dtype=torch.complex128, device=dev))
            else:
                if k:
                    for y in _quarters(W, g.q0, g.q1)[:3]:
                        y.zero_()
                _quarters(W, g.q0, g.q1)[3].mul_(np.exp(-1j * g.theta) * math.sqrt(P if k == 0 else 1.0 - P))
            parts.append(W)
        W = torch.cat(parts)
        m = W.shape[0]
        G = np.zeros((m, m), np.complex128)
        for i in range(m):
            for j in range(i, m):
                G[i, j] = complex(torch.vdot(W[i], W[j]))
                G[j, i] = np.conj(G[i, j])
        w, Q = np.linalg.eigh(G)
        w, Q = w[::-1], Q[:, ::-1]
        nz = int(np.sum(w > zero_tol * w[0]))
        keep = min(nz, r)
        if nz > r:
            while keep > 0 and w[keep - 1] - w[keep] <= 1e-9 * w[0]:
                keep -= 1
        kept = float(np.sum(w[:keep]))
        C = torch.as_tensor(np.ascontiguousarray(Q[:, :keep].T) / math.sqrt(kept), device=dev)
        V = torch.empty((keep, 1 << n), dtype=torch.complex128, device=dev)
        for c0 in range(0, 1 << n, 1 << 20):
            V[:, c0:c0 + (1 << 20)] = C @ W[:, c0:c0 + (1 << 20)]
        log_trace += math.log(kept)
    if case["circuit"] == "qft":
        # psi above carries its SWAPs as a relabelling; undo it to compare with the columns
        idx = torch.arange(1 << n, device=dev)
        src = torch.zeros_like(idx)
        for b in range(n):
            src |= ((idx >> b) & 1) << unused[b]
        psi = psi[:, src]
    fn = sum(abs(complex(torch.vdot(psi[0], V[c]))) ** 2 for c in range(V.shape[0]))
    return {"F": np.array([fn * math.exp(log_trace), fn, log_trace]), "ranks": None, "columns": None}


def _exact_gates(case, seed, dev):
    n = case["n"]
    gates, _, _ = _circuit(case, seed)
    psi = _random_state(n, case["dtype"], seed, dev).to(torch.complex128)[None].clone()
    ref = _random_state(n, case["dtype"], seed + 1, dev).to(torch.complex128)
    xi = _xi(seed, [g.site for g in gates], 1)[0]
    for g in gates:
        if g.kind == SWAP:
            x = _quarters(psi, g.q0, g.q1)
            t = x[1].clone()
            x[1].copy_(x[2])
            x[2].copy_(t)
        else:
            _evolve(psi, [g], list(range(n)), lambda h: np.array([h.e * xi[h.site]]) if h.noise else None)
    ov = complex(torch.vdot(psi[0], ref))
    na, nb = float(torch.linalg.vector_norm(psi[0])) ** 2, float(torch.linalg.vector_norm(ref)) ** 2
    return {"F": np.array([abs(ov) ** 2 / (na * nb), ov.real, ov.imag]), "psi": psi}


def exact(case, seed):
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    if case["kind"] in ("traj", "graph"):
        return _exact_traj(case, seed, dev)
    if case["kind"] in ("dm", "channels"):
        return _exact_dm(case, seed, dev)
    if case["kind"] == "fixed":
        return _exact_fixed(case, seed, dev)
    return _exact_gates(case, seed, dev)
