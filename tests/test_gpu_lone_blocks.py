"""A tiled plan's block on its own: the launch that the plan is priced for, a
dense block below 14 qubits in every precision, and the oracle's state."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20, sv.PREC_FP64: 2.0 ** -49}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("precision", list(STEP))
@pytest.mark.parametrize("n", [8, 10, 13, 14, 16])
def test_a_four_qubit_block_alone(n, precision):
    gates = [wc.Gate("MATRIX", (5, 1, 7, 2), (1,))]
    # the default prices, in place of what another test timed here: a one-block
    # pass 5 % below a dense block
    sv.set_cost_table(n, precision, np.array([0, 1, 1, 1, 1.02, 1.1, 1.6]))
    assert sv.fuse(to_binding(gates), n, 4, sv.RULE_AUTO, precision=precision).rule == (
        sv.RULE_TILED if n >= 14 else sv.RULE_ENHANCED)
    sv.stats_reset()
    sv.stats_enable(True)
    try:
        st = sv.State(n, "c128" if precision == sv.PREC_FP64 else "c64").set_basis(3)
        st.run(to_binding(gates), max_k=4, rule=sv.RULE_TILED, precision=precision)
        st.synchronize()
        tiles = sum(sv.stats_query(f, 1)[0] for f in sv.FAMILIES if f.startswith("tile"))
    finally:
        sv.stats_enable(False)
        sv.stats_reset()
    assert tiles == (n >= 14)
    start = np.zeros(1 << n, complex)
    start[3] = 1
    assert np.linalg.norm(st.read() - ref.simulate(n, gates, psi=start)) <= STEP[precision]
