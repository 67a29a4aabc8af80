"""Runs of a few small gates on both sides of the rule that lets them share a
pass (by their number, their qubits and the state's size), mixed with wider
blocks, against the oracle."""
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


@pytest.mark.parametrize("dtype,step", [("c64", 2.0 ** -21), ("c128", 2.0 ** -49)])
@pytest.mark.parametrize("n", [14, 19, 20])
def test_runs_of_a_few_gates(n, dtype, step):
    rng = np.random.default_rng(n)
    for count in (1, 2, 3, 4, 6, 12):
        for widest in (1, 2, 3):
            gates = []
            for i in range(count):
                k = int(rng.integers(1, widest + 1)) if i else widest
                gates.append(wc.Gate("MATRIX", tuple(int(q) for q in rng.choice(n, k, replace=False)), (i + 1,)))
            if count == 6:  # a wide block between two runs
                gates.insert(3, wc.Gate("MATRIX", tuple(int(q) for q in rng.choice(n, 5, replace=False)), (99,)))
            st = sv.State(n, dtype).set_product("+").run(to_binding(gates))
            assert np.linalg.norm(st.read() - ref.simulate(n, gates, "+")) <= len(gates) * step, (count, widest)
