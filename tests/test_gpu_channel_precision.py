"""The operators drawn in a trajectory are applied in the state's own FP32,
whatever the arithmetic of the gates, against the oracle: gates that a 16-bit
split leaves to the FP32 kernels follow channels on every qubit."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import density as dm
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("precision", [sv.PREC_FP32, sv.PREC_SPLIT_BF16, sv.PREC_SPLIT_FP16, sv.PREC_SPLIT_BF16X3])
@pytest.mark.parametrize("n", [9, 12, 15])
def test_operators_in_fp32(n, precision):
    rng = np.random.default_rng(n)
    first = [wc.Gate("RY", (q,), (0.4 + 0.1 * q,)) for q in range(n)]
    last = [wc.Gate("CZ", (0, 1)), wc.Gate("CZ", (n - 2, n - 1))]
    lib = [sv.amplitude_damping(q, 0.3, after=n) for q in range(n)]
    spots = [{"after": n, "left": [np.array(K) for K in op.left], "qubits": op.qubits} for op in lib]
    u = rng.random(n)
    st = sv.State(n, "c64")
    got = st.run(to_binding(first)).run_trajectory(to_binding(last), [op.at(0) for op in lib], u, max_k=4,
                                                   rule=sv.RULE_ENHANCED, precision=precision)
    want, picks = dm.trajectory(n, first + last, spots, u)
    assert [int(p) for p in got] == [int(p) for p in picks]
    # n gates, n operators and two sign changes, each rounding its matrix and the
    # result to 2^-24, the operators also in a fused pass of twice that
    assert np.linalg.norm(st.read() - want) <= (2 * n + 4 * n) * 2.0 ** -24
