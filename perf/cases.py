"""Performance cases of the state-vector framework.

Each case is one piece of work that a program using this package has it do, through the
public entry points (State, Plan, backward, Batch, DensityMatrix, ...), at sizes between a
launch-bound handful of qubits and the 30-qubit benchmark state:

  circuit      a random grid circuit started from a basis state (State.run with basis)
  gates        the same kind of circuit applied gate by gate (State.run's defaults)
  plan         a fused plan kept by the program and applied to the state it evolves
  gradient     energy and adjoint gradient of the hardware-efficient ansatz
  observables  norm, overlap, <H> and H|psi> of a state
  batch        noisy trajectories of uneven qubit counts, <Z_0> of each
  density      an exact density matrix under two-qubit depolarizing noise
  jumps        one trajectory with channels sampled on the pure state, then a measurement

The circuits are those of the benchmark: one-qubit layers drawn from sqrt(X), sqrt(Y),
sqrt(W) and fSim(pi/2, pi/6) on the four nearest-neighbour matchings of a grid.  Gate
choices, angles, noise draws, uniforms and state vectors come from the seed; sizes and the
shape of the grid come from the case.

Values that are computed from complex64 states and handed back in double precision
(gradients, <Z_0>) are returned as float32, the type a training loop keeps them in.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2111_06868_amd as sv

PRECISIONS = {"fp32": sv.PREC_FP32, "fp16": sv.PREC_SPLIT_FP16, "bf16": sv.PREC_SPLIT_BF16,
              "bf16x3": sv.PREC_SPLIT_BF16X3, "fp64": sv.PREC_FP64}
RULES = {"tiled": sv.RULE_TILED, "enhanced": sv.RULE_ENHANCED, "paper": sv.RULE_PAPER, "auto": sv.RULE_AUTO}
CHANNEL_KINDS = ("damping", "dephasing", "depolarizing")


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a small variational problem: every launch and every host call is latency
        {"name": "gradient10", "kind": "gradient", "n": 10, "layers": 4, "precision": "fp32"},
        # the smallest benchmark circuit (2 x 7 grid, 225 gates): a state that one compute unit's LDS holds
        {"name": "circuit14_fp16", "kind": "circuit", "n": 14, "cols": 7, "depth": 12, "dtype": "c64",
         "precision": "fp16", "rule": "tiled", "max_k": 4, "norm": False},
        # the benchmark's gradient: 708 gates, 480 angles, 39 Pauli terms
        {"name": "gradient20", "kind": "gradient", "n": 20, "layers": 12, "precision": "fp32"},
        # trajectories of the benchmark's range of sizes and depths
        {"name": "batch96", "kind": "batch", "count": 96, "n_min": 10, "n_max": 22, "depth_min": 8, "depth_max": 24,
         "p": 1e-3, "precision": "fp16"},
        # an odd number of qubits on a ladder with a missing site, in the default arithmetic
        {"name": "circuit23_fp32", "kind": "circuit", "n": 23, "cols": 12, "depth": 12, "dtype": "c64",
         "precision": "fp32", "rule": "tiled", "max_k": 4, "norm": True},
        # State.run as it is called with nothing but gates
        {"name": "gates24", "kind": "gates", "n": 24, "cols": 6, "depth": 8, "dtype": "c64"},
        # the exact density matrix of the noisy 3 x 4 grid circuit (a 24-qubit state) in the benchmark's arithmetic
        {"name": "density12_bf16x3", "kind": "density", "n": 12, "cols": 4, "depth": 12, "p": 1e-3, "dtype": "c64",
         "precision": "bf16x3", "rule": "tiled"},
        # amplitude damping on every qubit after every cycle, sampled on the pure state
        {"name": "jumps24", "kind": "jumps", "n": 24, "cols": 12, "depth": 4, "channel": "damping", "p": 0.01,
         "measured": 4, "dtype": "c64"},
        # the double-precision run that results are checked against
        {"name": "circuit25_fp64", "kind": "circuit", "n": 25, "cols": 5, "depth": 10, "dtype": "c128",
         "precision": "fp64", "rule": "tiled", "max_k": 4, "norm": True},
        # a plan of dense blocks that the program keeps and applies again and again
        {"name": "plan27_k5", "kind": "plan", "n": 27, "cols": 9, "depth": 8, "precision": "fp32",
         "rule": "enhanced", "max_k": 5},
        # what is read off a state: norm, overlap, <H> and H|psi> for the chain Hamiltonian
        {"name": "observables26", "kind": "observables", "n": 26, "strings": 8, "dtype": "c64"},
        # the headline: 5 x 6 grid, 845 gates, an 8 GiB state, restart, circuit and norm
        {"name": "circuit30_fp16", "kind": "circuit", "n": 30, "cols": 6, "depth": 20, "dtype": "c64",
         "precision": "fp16", "rule": "tiled", "max_k": 4, "norm": True},
    ]


def draw(rng):
    kind = rng.choice(("circuit", "circuit", "circuit", "gates", "plan", "gradient", "observables", "batch", "density",
                       "jumps"))
    if kind == "circuit":
        dtype = rng.choice(("c64", "c64", "c64", "c128"))
        n = rng.randint(8, 28 if dtype == "c64" else 26)
        precision = rng.choice(("fp16", "fp32", "bf16", "bf16x3")) if dtype == "c64" else "fp64"
        rule = rng.choice(("tiled", "tiled", "enhanced", "auto"))
        return {"kind": kind, "n": n, "cols": rng.randint(2, n), "depth": rng.randint(4, 16), "dtype": dtype,
                "precision": precision, "rule": rule, "max_k": -1 if rule == "auto" else 4,
                "norm": rng.random() < 0.5}
    if kind == "gates":
        dtype = rng.choice(("c64", "c128"))
        n = rng.randint(6, 26 if dtype == "c64" else 24)
        return {"kind": kind, "n": n, "cols": rng.randint(2, n), "depth": rng.randint(2, 8), "dtype": dtype}
    if kind == "plan":
        n = rng.randint(11, 27)
        rule = rng.choice(("enhanced", "paper"))
        return {"kind": kind, "n": n, "cols": rng.randint(2, n), "depth": rng.randint(2, 10),
                "precision": rng.choice(("fp32", "fp32", "fp16", "bf16")), "rule": rule, "max_k": rng.randint(2, 6)}
    if kind == "gradient":
        return {"kind": kind, "n": rng.randint(4, 21), "layers": rng.randint(1, 10),
                "precision": rng.choice(("fp32", "fp32", "fp16", "bf16x3"))}
    if kind == "observables":
        return {"kind": kind, "n": rng.randint(7, 27), "strings": rng.randint(0, 24), "dtype": rng.choice(("c64", "c64", "c128"))}
    if kind == "batch":
        lo = rng.randint(4, 16)
        return {"kind": kind, "count": int(math.exp(rng.uniform(math.log(4), math.log(96)))), "n_min": lo,
                "n_max": rng.randint(lo, 21), "depth_min": 4, "depth_max": rng.randint(6, 20), "p": 1e-3,
                "precision": rng.choice(("fp16", "fp32", "bf16", "bf16x3"))}
    if kind == "density":
        n = rng.randint(3, 12)
        dtype = rng.choice(("c64", "c64", "c64", "c128"))
        return {"kind": kind, "n": n, "cols": rng.randint(2, n), "depth": rng.randint(2, 10), "p": rng.choice((1e-3, 1e-2)),
                "dtype": dtype, "precision": rng.choice(("bf16x3", "bf16", "fp32")) if dtype == "c64" else "fp64",
                "rule": rng.choice(("tiled", "tiled", "enhanced"))}
    n = rng.randint(8, 24)
    return {"kind": kind, "n": n, "cols": rng.randint(2, n), "depth": rng.randint(1, 4), "channel": rng.choice(CHANNEL_KINDS),
            "p": rng.choice((0.01, 0.1)), "measured": rng.randint(1, 8), "dtype": rng.choice(("c64", "c64", "c128"))}


# ------------------------------------------------------------------ circuits
def grid_gates(n, cols, depth, rng):
    """Random circuit on n sites, row by row on a grid of `cols` columns (the last row may be short), as
    (name, qubits, params) tuples; also the positions in the list where a cycle's fSims end."""
    at = [(q // cols, q % cols) for q in range(n)]
    matchings = [[], [], [], []]
    for q, (r, c) in enumerate(at):
        if c + 1 < cols and q + 1 < n:
            matchings[0 if (r + c) % 2 == 0 else 1].append((q, q + 1))
        if q + cols < n:
            matchings[2 if (r + c) % 2 == 0 else 3].append((q, q + cols))
    names = ("SQRT_X", "SQRT_Y", "SQRT_W")
    gates, ends, last = [], [], [-1] * n
    for cycle in range(depth):
        for q in range(n):
            last[q] = int(rng.choice([i for i in range(3) if i != last[q]]))
            gates.append((names[last[q]], (q,), ()))
        gates += [("FSIM", edge, (math.pi / 2, math.pi / 6)) for edge in matchings[cycle % 4]]
        ends.append(len(gates))
    return gates, ends


def trajectory_sizes(case):
    """Qubit counts and depths of a batch: fixed by the case, so that every seed asks for the same work."""
    rng = np.random.default_rng([case["count"], case["n_min"], case["n_max"], case["depth_max"]])
    return [(int(rng.integers(case["n_min"], case["n_max"] + 1)), int(rng.integers(case["depth_min"], case["depth_max"] + 1)))
            for _ in range(case["count"])]


def trajectories(case, seed):
    """Ladder circuits with Pauli strings inserted after the fSims with probability p."""
    out = []
    for t, (n, depth) in enumerate(trajectory_sizes(case)):
        rng = np.random.default_rng([seed, t])
        gates = []
        for g in grid_gates(n, (n + 1) // 2, depth, rng)[0]:
            gates.append(g)
            if g[0] == "FSIM" and rng.random() < case["p"]:
                gates += [("IXYZ"[d], (q,), ()) for q, d in zip(g[1], divmod(int(rng.integers(16)), 4)) if d]
        out.append((n, gates))
    return out


def ansatz(n, layers, rng):
    """RY and RZ on every qubit, then CZ along the chain, per layer: (name, qubits, params, param_index)."""
    gates = []
    for layer in range(layers):
        for j, name in enumerate(("RY", "RZ")):
            gates += [(name, (q,), (float(rng.uniform(0, 2 * math.pi)),), (2 * layer + j) * n + q) for q in range(n)]
        gates += [("CZ", (q, q + 1)) for q in range(n - 1)]
    return gates


def chain(n):
    """sum_i Z_i Z_{i+1} + 0.5 sum_i X_i."""
    return [(1.0, ((i, "Z"), (i + 1, "Z"))) for i in range(n - 1)] + [(0.5, ((i, "X"),)) for i in range(n)]


def hamiltonian(case, seed):
    """The chain and `strings` random Pauli strings of up to four factors."""
    rng = np.random.default_rng([seed, 1])
    terms = chain(case["n"])
    for _ in range(case["strings"]):
        qs = rng.choice(case["n"], size=int(rng.integers(1, 5)), replace=False)
        terms.append((float(rng.normal()), tuple((int(q), "XYZ"[int(rng.integers(3))]) for q in qs)))
    return terms


def channel_spots(case, gates, ends):
    """(after, qubits) of the channels: on every qubit, or on every fSim's pair, after each cycle."""
    if case["channel"] != "depolarizing":
        return [(a, (q,)) for a in ends for q in range(case["n"])]
    begins = [0] + ends[:-1]
    return [(a, g[1]) for b, a in zip(begins, ends) for g in gates[b:a] if g[0] == "FSIM"]


def random_state(n, dtype, seed, into=None):
    """A normalised state with Gaussian amplitudes, as interleaved (re, im)."""
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    real = torch.float32 if dtype == "c64" else torch.float64
    v = torch.randn(2 << n, dtype=real, device="cuda", generator=gen) * math.sqrt(0.5 / (1 << n))
    if into is None:
        return v
    into.copy_(v)
    return into


# ------------------------------------------------------------------ what a program holds, and one pass
def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    rng = np.random.default_rng(seed)
    if kind in ("circuit", "gates"):
        s["gates"] = sv.GateArray(grid_gates(case["n"], case["cols"], case["depth"], rng)[0])
        s["psi"] = sv.State(case["n"], case["dtype"])
    elif kind == "plan":
        gates = grid_gates(case["n"], case["cols"], case["depth"], rng)[0]
        s["precision"] = PRECISIONS[case["precision"]]
        s["plan"] = sv.fuse(gates, case["n"], case["max_k"], RULES[case["rule"]], precision=s["precision"])
        s["psi"] = sv.State(case["n"], "c64")
        random_state(case["n"], "c64", seed, s["psi"].tensor)
    elif kind == "gradient":
        s["gates"] = sv.GateArray(ansatz(case["n"], case["layers"], rng))
        s["H"] = sv.pauli_sum(chain(case["n"]))
        s["psi"], s["scratch"] = sv.State(case["n"], "c64"), sv.State(case["n"], "c64")
    elif kind == "observables":
        s["psi"], s["phi"], s["out"] = (sv.State(case["n"], case["dtype"]) for _ in range(3))
        random_state(case["n"], case["dtype"], seed, s["psi"].tensor)
        random_state(case["n"], case["dtype"], seed + 1, s["phi"].tensor)
        s["H"] = sv.pauli_sum(hamiltonian(case, seed))
    elif kind == "batch":
        s["batch"] = sv.Batch(trajectories(case, seed), max_k=4, precision=PRECISIONS[case["precision"]])
    elif kind == "density":
        gates = grid_gates(case["n"], case["cols"], case["depth"], rng)[0]
        s["gates"] = sv.GateArray(gates)
        s["ops"] = [sv.depolarizing(g[1], case["p"], after=i + 1) for i, g in enumerate(gates) if g[0] == "FSIM"]
        s["rho"] = sv.DensityMatrix(case["n"], case["dtype"])
        s["H"] = sv.pauli_sum(chain(case["n"]))
    else:
        gates, ends = grid_gates(case["n"], case["cols"], case["depth"], rng)
        make = {"damping": lambda q, a: sv.amplitude_damping(q[0], case["p"], after=a),
                "dephasing": lambda q, a: sv.dephasing(q[0], case["p"], "X", after=a),
                "depolarizing": lambda q, a: sv.depolarizing(q, case["p"], after=a)}[case["channel"]]
        s["gates"] = sv.GateArray(gates)
        s["ops"] = [make(q, a) for a, q in channel_spots(case, gates, ends)]
        s["uniforms"] = rng.random(len(s["ops"]))
        s["measured"] = tuple(range(case["n"]))[-case["measured"]:]
        s["draws"] = rng.random(case["measured"])
        s["psi"] = sv.State(case["n"], case["dtype"])
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "circuit":
        psi = s["psi"].run(s["gates"], max_k=case["max_k"], rule=RULES[case["rule"]],
                           precision=PRECISIONS[case["precision"]], basis=0)
        out = {"state": psi.tensor}
        if case["norm"]:
            out["norm"] = psi.norm2()
        return out
    if kind == "gates":
        return {"state": s["psi"].set_basis(0).run(s["gates"]).tensor}
    if kind == "plan":
        return {"state": s["psi"].apply_plan(s["plan"], precision=s["precision"]).tensor}
    if kind == "gradient":
        precision = PRECISIONS[case["precision"]]
        psi = s["psi"].set_basis(0).run(s["gates"], max_k=-1, rule=sv.RULE_AUTO, precision=precision)
        energy = psi.expectation(s["H"])
        grad = sv.backward(psi, s["scratch"], s["gates"], s["H"], 2 * case["n"] * case["layers"], precision=precision)
        return {"energy": energy, "grad": grad.astype(np.float32)}
    if kind == "observables":
        psi = s["psi"]
        overlap = psi.inner(s["phi"])
        return {"norm": psi.norm2(), "overlap": [overlap.real, overlap.imag], "energy": psi.expectation(s["H"]),
                "h_psi": psi.apply_pauli_sum(s["H"], s["out"]).tensor}
    if kind == "batch":
        return {"z0": s["batch"].run(use_graph=True).astype(np.float32)}
    if kind == "density":
        rho = s["rho"].set_basis(0).run(s["gates"], s["ops"], max_k=4, rule=RULES[case["rule"]],
                                        precision=PRECISIONS[case["precision"]])
        return {"rho": rho.state.tensor, "energy": rho.expectation(s["H"])}
    psi = s["psi"].set_basis(0)
    picks = psi.run_trajectory(s["gates"], s["ops"], s["uniforms"], max_k=4, rule=sv.RULE_TILED)
    bits, p = psi.measure(s["measured"], s["draws"])
    return {"state": psi.tensor, "picks": picks, "bits": [int(b) for b in bits], "p": p}


# ------------------------------------------------------------------ what a pass cannot do without
def gate_flops(gates, n):
    """Dense k-qubit products on 2^n amplitudes: 2^k complex multiply-adds an amplitude."""
    return sum(8.0 * (1 << len(g[1])) for g in gates) * (1 << n)


def work(case):
    kind, n = case["kind"], case.get("n", 0)
    rng = np.random.default_rng(0)
    amp = 16 if case.get("dtype") == "c128" else 8
    if kind in ("circuit", "gates"):  # the state is written; nothing of it is read
        return {"bytes": amp << n, "flops": gate_flops(grid_gates(n, case["cols"], case["depth"], rng)[0], n)}
    if kind == "plan":
        return {"bytes": 2 * (8 << n), "flops": gate_flops(grid_gates(n, case["cols"], case["depth"], rng)[0], n)}
    if kind == "gradient":  # forward, then two states swept back; the gradient is what is written
        gates = ansatz(n, case["layers"], rng)
        return {"bytes": 24.0 * len(gates) + 8.0 * 2 * n * case["layers"], "flops": 3 * gate_flops(gates, n)}
    if kind == "observables":  # psi and phi read, H psi written
        return {"bytes": 3 * (amp << n), "flops": (8.0 * 2 + 16.0 * (2 * n - 1 + case["strings"])) * (1 << n)}
    if kind == "batch":
        sizes = trajectory_sizes(case)
        flops = sum(gate_flops(grid_gates(m, (m + 1) // 2, d, rng)[0], m) for m, d in sizes)
        return {"bytes": float(sum(8 << m for m, _ in sizes)), "flops": flops}  # every state can be read afterwards
    gates, ends = grid_gates(n, case["cols"], case["depth"], rng)
    if kind == "density":
        pairs = sum(1 for g in gates if g[0] == "FSIM")
        return {"bytes": amp << (2 * n), "flops": 2 * gate_flops(gates, 2 * n) + pairs * 8.0 * 16 * (1 << (2 * n))}
    spots = channel_spots(case, gates, ends)
    return {"bytes": amp << n, "flops": gate_flops(gates + [("K", q) for _, q in spots], n)}


# ------------------------------------------------------------------ the same in 64 bits, with plain torch
S2 = math.sqrt(0.5)
PAULI = {"I": np.eye(2), "X": np.array([[0, 1], [1, 0]]), "Y": np.array([[0, -1j], [1j, 0]]), "Z": np.diag([1, -1])}


def matrix(g):
    """Matrix of a gate tuple; the first qubit is the most significant bit of the local index."""
    name, p = g[0], g[2] if len(g) > 2 else ()
    if name in PAULI:
        return PAULI[name].astype(complex)
    if name.startswith("SQRT_"):
        P = {"X": PAULI["X"], "Y": PAULI["Y"], "W": S2 * (PAULI["X"] + PAULI["Y"])}[name[5:]]
        return 0.5 * ((1 + 1j) * PAULI["I"] + (1 - 1j) * P)
    if name in ("RX", "RY", "RZ"):
        return math.cos(p[0] / 2) * PAULI["I"] - 1j * math.sin(p[0] / 2) * PAULI[name[1]]
    if name == "CZ":
        return np.diag([1, 1, 1, -1]).astype(complex)
    m = np.zeros((4, 4), complex)  # FSIM
    m[0, 0], m[3, 3] = 1, np.exp(-1j * p[1])
    m[1, 1] = m[2, 2] = math.cos(p[0])
    m[1, 2] = m[2, 1] = -1j * math.sin(p[0])
    return m


def apply(psi, n, U, qubits):
    """U on the qubits (positions) of a complex128 vector."""
    k = len(qubits)
    shape, axis, top = [], {}, n
    for q in sorted(qubits, reverse=True):
        shape += [1 << (top - 1 - q), 2]
        axis[q] = len(shape) - 1
        top = q
    shape.append(1 << top)
    front = [axis[q] for q in qubits]
    perm = front + [i for i in range(len(shape)) if i not in front]
    x = psi.view(shape).permute(perm)
    mid = x.shape
    y = torch.matmul(torch.as_tensor(U, dtype=torch.complex128, device=psi.device), x.reshape(1 << k, -1))
    back = [perm.index(i) for i in range(len(perm))]
    return y.view(mid).permute(back).reshape(-1)


def apply_all(psi, n, gates):
    """The gates in order, one-qubit gates multiplied into the next two-qubit gate on their qubit."""
    held = {}
    for g in gates:
        U = matrix(g)
        if len(g[1]) == 1:
            held[g[1][0]] = U @ held.get(g[1][0], np.eye(2))
        else:
            a, b = (held.pop(q, np.eye(2)) for q in g[1])
            psi = apply(psi, n, U @ np.kron(a, b), g[1])
    for q, U in held.items():
        psi = apply(psi, n, U, (q,))
    return psi


def zero_state(n):
    psi = torch.zeros(1 << n, dtype=torch.complex128, device="cuda")
    psi[0] = 1
    return psi


def reals(psi):
    return torch.view_as_real(psi).reshape(-1)


def times_h(psi, n, terms):
    out = torch.zeros_like(psi)
    for c, factors in terms:
        v = psi
        for q, p in factors:
            v = apply(v, n, PAULI[p], (q,))
        out += c * v
    return out


def kraus(case, k):
    """The operators of the sampled channel."""
    p = case["p"]
    if case["channel"] == "damping":
        return [np.diag([1, math.sqrt(1 - p)]).astype(complex), np.array([[0, math.sqrt(p)], [0, 0]], complex)]
    if case["channel"] == "dephasing":
        return [math.sqrt(1 - p) * PAULI["I"].astype(complex), math.sqrt(p) * PAULI["X"].astype(complex)]
    return depolarizing(p)


def depolarizing(p):
    weights = [1 - p + p / 16] + [p / 16] * 15
    return [math.sqrt(w) * np.kron(PAULI["IXYZ"[i // 4]], PAULI["IXYZ"[i % 4]]) for i, w in enumerate(weights)]


def sampled(psi, n, ops, qubits, u):
    """K_i psi / |K_i psi|, the first operator whose running weight passes u of the sum."""
    weights = [float(torch.linalg.vector_norm(apply(psi, n, K, qubits)) ** 2) for K in ops]
    total, so_far, pick = sum(weights), 0.0, -1
    for i, w in enumerate(weights):
        so_far += w
        if w > 0:
            pick = i
            if u * total < so_far:
                break
    return apply(psi, n, ops[pick] / math.sqrt(weights[pick]), qubits), pick, weights[pick] / total


def exact(case, seed):
    kind, n = case["kind"], case.get("n", 0)
    rng = np.random.default_rng(seed)
    if kind in ("circuit", "gates", "plan"):
        gates = grid_gates(n, case["cols"], case["depth"], rng)[0]
        if kind == "plan":
            psi = torch.view_as_complex(random_state(n, "c64", seed).double().view(-1, 2))
        else:
            psi = zero_state(n)
        out = {"state": reals(apply_all(psi, n, gates))}
        if case.get("norm"):
            out["norm"] = 1.0
        return out
    if kind == "gradient":
        gates, terms = ansatz(n, case["layers"], rng), chain(n)
        phi = apply_all(zero_state(n), n, gates)
        lam = times_h(phi, n, terms)
        grad = np.zeros(2 * n * case["layers"])
        energy = float(torch.vdot(phi, lam).real)
        for g in reversed(gates):
            if g[0] != "CZ":
                grad[g[3]] += float(torch.vdot(lam, apply(phi, n, PAULI[g[0][1]], g[1])).imag)
            back = matrix(g).conj().T
            phi, lam = apply(phi, n, back, g[1]), apply(lam, n, back, g[1])
        return {"energy": energy, "grad": grad}
    if kind == "observables":
        psi, phi = (torch.view_as_complex(random_state(n, case["dtype"], seed + k).double().view(-1, 2)) for k in (0, 1))
        hpsi, overlap = times_h(psi, n, hamiltonian(case, seed)), torch.vdot(psi, phi)
        return {"norm": float(torch.vdot(psi, psi).real), "overlap": [float(overlap.real), float(overlap.imag)],
                "energy": float(torch.vdot(psi, hpsi).real), "h_psi": reals(hpsi)}
    if kind == "batch":
        z0 = []
        for m, gates in trajectories(case, seed):
            w = apply_all(zero_state(m), m, gates).abs().square()
            z0.append(float(w[0::2].sum() - w[1::2].sum()))
        return {"z0": np.array(z0)}
    if kind == "density":  # the vector of 2n qubits with U on the row index and conj(U) on the column index
        rho = zero_state(2 * n)
        channel = sum(np.kron(K, K.conj()) for K in depolarizing(case["p"]))
        for g in grid_gates(n, case["cols"], case["depth"], rng)[0]:
            row = tuple(q + n for q in g[1])
            U = matrix(g)
            full = np.kron(U, U.conj())
            if g[0] == "FSIM":
                full = channel @ full
            rho = apply(rho, 2 * n, full, row + tuple(g[1]))
        d = 1 << n
        energy = 0.0
        for c, factors in chain(n):  # Tr(P rho)
            v = rho
            for q, p in factors:
                v = apply(v, 2 * n, PAULI[p], (q + n,))
            energy += c * float(v.view(d, d).diagonal().sum().real)
        return {"rho": reals(rho), "energy": energy}
    gates, ends = grid_gates(n, case["cols"], case["depth"], rng)
    spots = channel_spots(case, gates, ends)
    uniforms, draws = rng.random(len(spots)), rng.random(case["measured"])
    psi, done, picks, bits, p = zero_state(n), 0, [], [], 1.0
    for (after, qubits), u in zip(spots, uniforms):
        psi = apply_all(psi, n, gates[done:after])
        done = after
        psi, pick, _ = sampled(psi, n, kraus(case, len(qubits)), qubits, u)
        picks.append(pick)
    psi = apply_all(psi, n, gates[done:])
    ends = [np.diag([1, 0]).astype(complex), np.diag([0, 1]).astype(complex)]
    for q, u in zip(range(n - case["measured"], n), draws):
        psi, bit, w = sampled(psi, n, ends, (q,), u)
        bits.append(bit)
        p *= w
    return {"state": reals(psi), "picks": np.array(picks, dtype=np.int32), "bits": bits, "p": p}
