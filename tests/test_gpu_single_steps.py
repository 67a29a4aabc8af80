"""Steps of one qubit with parameters whose gates lie on at most three qubits:
the sums and the undoing of the gates in one launch, against parameter shifts
of the oracle; every position of the qubit in the block, low and high."""
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
@pytest.mark.parametrize("n", [1, 2, 3, 5, 11, 13, 15])
def test_one_launch_a_step(n, dtype, tol):
    rng = np.random.default_rng(n)
    k = min(n, 3)
    gates, widths = [], []
    for p in range(9):
        qs = [int(q) for q in rng.choice(n, k, replace=False)] if p else list(range(n))[-k:]
        kind = ("RX", "RY", "RZ")[p % 3]
        wide = min(k, 1 + p % 3)
        if n == 1:
            gates.append(wc.Gate("MATRIX", (0,), (p,)))
        else:
            gates += [wc.Gate("FSIM", (qs[0], qs[1]), (1.1, 0.3)), wc.Gate("MATRIX", tuple(qs[:max(2, wide)]), (p,))]
        gates.append(wc.Gate(kind, (qs[0],), (float(rng.uniform(0, 6)),), p))
    H = [(1.0, ((0, "Z"),)), (0.5, ((n - 1, "X"),)), (0.25, tuple((q, "Y") for q in range(k)))]
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    psi.set_product("+").run(to_binding(gates), max_k=4, rule=sv.RULE_ENHANCED)
    sv.stats_reset()
    sv.stats_enable(True)
    try:
        got = sv.backward(psi, lam, to_binding(gates), H, 9)
        launches = [sv.stats_query("adjoint", j)[0] for j in range(4)]
        other = sum(sv.stats_query(f, j)[0] for f in sv.FAMILIES if f not in ("adjoint", "reduce") for j in range(1, 17))
    finally:
        sv.stats_enable(False)
        sv.stats_reset()
    if n > 1:  # a step undoes its rotation and the gates before it
        assert sum(launches) == 9 and other == 0
    for p in range(9):
        i = next(i for i, g in enumerate(gates) if g.param_index == p)
        e = []
        for s in (1, -1):
            shifted = list(gates)
            shifted[i] = wc.Gate(gates[i].name, gates[i].qubits, (gates[i].params[0] + s * np.pi / 2,), p)
            e.append(ref.expectation(ref.simulate(n, shifted, "+"), H))
        # two sweeps, two states, |H| <= 1.75
        assert abs(got[p] - 0.5 * (e[0] - e[1])) <= 4 * len(gates) * tol * 1.75, p
