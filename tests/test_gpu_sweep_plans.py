"""Sweeps whose steps share plans: runs of the same positions one after another
with other angles and kinds, then of other positions, few steps and many
(planned by several threads), against parameter shifts of the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("dtype,tol", [("c64", 2.0 ** -21), ("c128", 2.0 ** -49)])
@pytest.mark.parametrize("n,layers", [(3, 1), (5, 6), (11, 24)])
def test_steps_of_equal_and_other_positions(n, layers, dtype, tol):
    rng = np.random.default_rng(n)
    gates, params = [wc.Gate("H", (q,)) for q in range(n)], 0
    for layer in range(layers):
        qs = list(range(n)) if layer % 5 < 3 else [int(q) for q in rng.permutation(n)]
        kind = ("RX", "RY", "RZ")[int(rng.integers(3))]
        for q in qs:
            gates.append(wc.Gate(kind, (q,), (float(rng.uniform(0, 6)),), params))
            params += 1
        gates += [wc.Gate(("CZ", "CX")[layer % 2], (a, b)) for a, b in zip(qs, qs[1:])]
    H = [(1.0, ((0, "Z"),)), (0.5, ((1, "X"), (n - 1, "Z")))]
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    psi.set_basis(0).run(to_binding(gates), max_k=4, rule=sv.RULE_ENHANCED)
    got = sv.backward(psi, lam, to_binding(gates), H, params)
    for p in (range(params) if params < 40 else rng.choice(params, 12, replace=False)):
        i = next(i for i, g in enumerate(gates) if g.param_index == p)
        e = []
        for s in (1, -1):
            shifted = list(gates)
            shifted[i] = wc.Gate(gates[i].name, gates[i].qubits, (gates[i].params[0] + s * np.pi / 2,), p)
            e.append(ref.expectation(ref.simulate(n, shifted, "0"), H))
        assert abs(got[p] - 0.5 * (e[0] - e[1])) <= 4 * len(gates) * tol * 1.5, p  # two sweeps, two states, |H| <= 1.5
