"""Adjoint gradients of runs of one-qubit gates (several rotations and fixed
gates on a qubit share one pass of transition sums) against the parameter
shift of the oracle, from one qubit to more than a workgroup's qubits."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from oracle import ref
from workloads import circuits as wc
from helpers import to_binding

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _circuit(n, rng):
    """Rotations in runs of mixed length; two rotations share parameter 0."""
    gates, p = [], 0
    for layer in range(3):
        for _ in range(2 * n + 3):
            q = int(rng.integers(n))
            name = ("RX", "RY", "RZ", "H", "SQRT_W")[int(rng.integers(5))]
            if name[0] == "R":
                gates.append(wc.Gate(name, (q,), (float(rng.uniform(0, 6)),), 0 if rng.random() < 0.1 else p))
                p += gates[-1].param_index == p
            else:
                gates.append(wc.Gate(name, (q,)))
        for q in range(layer % 2, n - 1, 2):
            gates.append(wc.Gate("FSIM", (q + 1, q), (0.7, 0.3)))
    gates.append(wc.Gate("CZ", (0, n - 1)) if n > 1 else wc.Gate("H", (0,)))
    return gates, p


@pytest.mark.parametrize("n", [1, 2, 3, 5, 9, 11, 12, 14])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_runs_against_parameter_shift(n, dtype):
    rng = np.random.default_rng(n)
    gates, count = _circuit(n, rng)
    H = [(1.0, ((q, "Z"),)) for q in range(n)] + [(0.5, ((q, "X"), (q + 1, "Y"))) for q in range(n - 1)]
    psi = sv.State(n, dtype).run(to_binding(gates), max_k=4, rule=sv.RULE_ENHANCED)
    got = sv.backward(psi, sv.State(n, dtype), to_binding(gates), H, count)
    # single gates shifted one at a time (parameters may be shared)
    picked = [i for i, g in enumerate(gates) if g.param_index >= 0]
    want, seen = np.zeros(count), {}
    for p in sorted({gates[i].param_index for i in picked})[:: max(1, count // 8)]:
        seen[p] = 0.0
        for i in picked:
            if gates[i].param_index != p:
                continue
            e = []
            for s in (1, -1):
                shifted = list(gates)
                g = gates[i]
                shifted[i] = wc.Gate(g.name, g.qubits, (g.params[0] + s * np.pi / 2,), g.param_index)
                e.append(ref.expectation(ref.simulate(n, shifted, "0"), H))
            seen[p] += 0.5 * (e[0] - e[1])
    size = sum(abs(c) for c, _ in H)
    # each of some 40 fused blocks of the two sweeps rounds a norm-1 vector;
    # lam has norm at most sum |c|
    tol = 2 * 80 * 2.0 ** (-24 if dtype == "c64" else -50) * size
    for p, w in seen.items():
        assert abs(got[p] - w) <= tol, (p, got[p], w)
    psi_back = psi.read()  # the sweep ends at the initial state
    assert abs(abs(psi_back[0]) - 1.0) <= 80 * 2.0 ** -22
