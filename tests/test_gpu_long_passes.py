"""Passes long enough to spread their workgroups' starts (more than 16 tiles a
workgroup) in every kind of tile pass, against single blocks in FP64."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20, sv.PREC_SPLIT_BF16: 2.0 ** -15, sv.PREC_FP64: 2.0 ** -49}
N = 27


def _gates():
    rng = np.random.default_rng(1)
    gates = []
    for layer in range(2):
        gates += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(N)]
        gates += [wc.Gate("FSIM", (q, q + 1), (1.1, 0.3)) for q in range(layer % 2, N - 1, 2)]
    return to_binding(gates)


@pytest.fixture(scope="module")
def want():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    plan = sv.fuse(_gates(), N, 3, sv.RULE_ENHANCED, precision=sv.PREC_FP64).own_blocks()
    st = sv.State(N, "c128").set_basis(0).apply_plan(plan, precision=sv.PREC_FP64)
    yield st
    st.free()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("rule,precision", [(sv.RULE_TILED, p) for p in STEP] +
                         [(sv.RULE_NONE, sv.PREC_FP32), (sv.RULE_NONE, sv.PREC_FP64)])
def test_27_qubits(want, rule, precision):
    import torch
    gates = _gates()
    st = sv.State(N, "c128" if precision == sv.PREC_FP64 else "c64").set_basis(0)
    st.run(gates, max_k=4, rule=rule, precision=precision)
    st.synchronize()
    want.synchronize()
    got, ref = st.tensor.view(-1), want.tensor.view(-1)
    err = sum(float((g.double() - r).square().sum()) for g, r in zip(got.split(1 << 25), ref.split(1 << 25))) ** 0.5
    assert err <= len(gates) * STEP[precision]
    del got, ref
    st.free()
    torch.cuda.empty_cache()
