"""Plans of the paper and enhanced rules whose dense blocks run as tile passes
(from 14 qubits on) against the oracle: every precision, a gate wider than a
tile block, a plan kept for a larger state or applied in another precision,
captured and from a basis state."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state: 32-term FP32 (FP64) sums, the
# BF16 split's dropped 2^-17 terms
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20,
        sv.PREC_SPLIT_BF16: 2.0 ** -15, sv.PREC_FP64: 2.0 ** -49}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _circuit(n, wide, rng):
    gates = []
    for layer in range(4):
        gates += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(n)]
        gates += [wc.Gate("FSIM", (q + 1, q), (1.1, 0.4)) for q in range(layer % 2, n - 1, 2)]
        gates.append(wc.Gate("FSIM", (0, n - 1), (0.3, 0.9)))
        if wide:
            gates.append(wc.Gate("MATRIX", tuple(int(q) for q in rng.choice(n, wide, replace=False)), (layer + 1,)))
    return gates


@pytest.mark.parametrize("n", [13, 14, 15, 18])
@pytest.mark.parametrize("rule,max_k,wide", [(sv.RULE_PAPER, 4, 0), (sv.RULE_PAPER, 6, 4), (sv.RULE_ENHANCED, 4, 3),
                                             (sv.RULE_ENHANCED, 5, 5), (sv.RULE_ENHANCED, 5, 0)])
@pytest.mark.parametrize("precision", list(STEP))
def test_against_oracle(n, rule, max_k, wide, precision):
    gates = _circuit(n, wide, np.random.default_rng(n + max_k))
    bound = to_binding(gates)
    dtype = "c128" if precision == sv.PREC_FP64 else "c64"
    want = ref.simulate(n, gates, "0")
    tol = len(gates) * STEP[precision]
    runs = {"run": sv.State(n, dtype).run(bound, max_k=max_k, rule=rule, precision=precision, basis=0),
            "graph": sv.State(n, dtype).run(bound, max_k=max_k, rule=rule, precision=precision, use_graph=True)}
    other = sv.PREC_FP64 if precision != sv.PREC_FP64 else sv.PREC_FP32
    for name, p in (("plan", sv.fuse(bound, n, max_k, rule, precision=precision)), ("any", sv.fuse(bound, n, max_k, rule)),
                    ("other", sv.fuse(bound, n, max_k, rule, precision=other))):
        runs[name] = sv.State(n, dtype).apply_plan(p, precision=precision)
    for name, st in runs.items():
        assert np.linalg.norm(st.read() - want) <= tol, name


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_plan_on_a_larger_state(dtype):
    n, gates = 14, _circuit(14, 0, np.random.default_rng(0))
    plan = sv.fuse(to_binding(gates), n, 5, sv.RULE_ENHANCED)
    got = sv.State(16, dtype).set_basis(3 << 14).apply_plan(plan).read()
    want = ref.simulate(n, gates, "0")
    assert np.linalg.norm(got[3 << 14:] - want) <= len(gates) * STEP[sv.PREC_FP32 if dtype == "c64" else sv.PREC_FP64]
    assert not got[:3 << 14].any()
