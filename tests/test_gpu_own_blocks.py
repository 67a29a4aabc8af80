"""Plans asked to apply their own blocks: a launch for each, of the block's own
kernel, and the oracle's state; without the request they share passes."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20, sv.PREC_FP64: 2.0 ** -49}
DENSE = {sv.PREC_FP32: ("mfma_f32", "reg"), sv.PREC_SPLIT_FP16: ("split_fp16",), sv.PREC_FP64: ("generic", "reg")}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _launches(plan, n, precision):
    sv.stats_reset()
    sv.stats_enable(True)
    try:
        st = sv.State(n, "c128" if precision == sv.PREC_FP64 else "c64").apply_plan(plan, precision=precision)
        st.synchronize()
        count = {(f, k): sv.stats_query(f, k)[0] for f in sv.FAMILIES for k in range(1, 17)}
    finally:
        sv.stats_enable(False)
        sv.stats_reset()
    return st.read(), count


@pytest.mark.parametrize("rule,max_k", [(sv.RULE_PAPER, 5), (sv.RULE_ENHANCED, 4), (sv.RULE_NONE, 6)])
@pytest.mark.parametrize("precision", list(STEP))
def test_a_launch_for_each_block(rule, max_k, precision):
    n = 15
    gates = wc.random_gate_list(n, 60, np.random.default_rng(max_k), max_k=2)
    want, tol = ref.simulate(n, gates, "0"), len(gates) * STEP[precision]
    plan = sv.fuse(to_binding(gates), n, max_k, rule, precision=precision)
    sizes = np.bincount([len(b.qubits) for b in plan.blocks(False)], minlength=7)
    got, count = _launches(plan.own_blocks(), n, precision)
    assert np.linalg.norm(got - want) <= tol
    for k in range(1, 7):
        own = DENSE[precision] if k >= 4 else ("reg",)
        assert sum(count[f, k] for f in own) == sizes[k], k
    assert sum(v for (f, _), v in count.items() if f.startswith("tile")) == 0
    got, _ = _launches(plan.own_blocks(False), n, precision)
    assert np.linalg.norm(got - want) <= tol
