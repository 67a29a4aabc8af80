"""Channels drawn together from one pass of joint probabilities
(sv_run_trajectory, sv_measure) against the oracle, which draws and applies
them one at a time: more qubits than one pass holds, several passes with
weights of operators not yet applied, multi-qubit channels with and without
constant weights, repeated qubits, channels that need their own pass, states
smaller than a tile and larger, and the rules their gates run under."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from oracle import density as dm
from oracle import ops as oracle_ops
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


def _ops(n, G, rng):
    """A mixed list of channels: the library's operators, the oracle's, uniforms."""
    lib, spots = [], []

    def add(op):
        lib.append(op)
        spots.append({"after": op.after, "left": [np.array(K) for K in op.left], "qubits": op.qubits})

    mid = G // 2
    for q in range(n):
        add(sv.amplitude_damping(q, 0.3, after=mid))
    for q in range(0, n - 1, 2):  # constant weights, distinct qubits
        add(sv.depolarizing((q, q + 1), 0.4, after=mid))
    # diagonal weights that are no product over the two qubits, then the same qubits again
    K0 = np.diag([1.0, 0.6, 0.8, 0.1])
    K1 = np.diag(np.sqrt(1 - np.diag(K0) ** 2))
    add(sv.SuperOp((n - 1, 0), left=[K0, K1], after=mid))
    add(sv.dephasing(0, 0.5, "Y", after=mid))
    add(sv.SuperOp((1, n - 2), left=wc.random_kraus_from_seed(7, 2, 3), after=mid))  # needs its own pass
    for q in range(n):
        add(sv.amplitude_damping(q, 0.2, 0.1, after=G))
    return lib, spots, rng.random(len(lib))


@pytest.mark.parametrize("n,dtype,rule,precision", [
    (4, "c64", sv.RULE_NONE, sv.PREC_FP32), (10, "c64", sv.RULE_ENHANCED, sv.PREC_FP32),
    (11, "c128", sv.RULE_PAPER, sv.PREC_FP64), (12, "c64", sv.RULE_AUTO, sv.PREC_FP32),
    (14, "c64", sv.RULE_TILED, sv.PREC_SPLIT_FP16), (15, "c128", sv.RULE_TILED, sv.PREC_FP64),
    (16, "c64", sv.RULE_TILED, sv.PREC_SPLIT_BF16X3)])
def test_grouped_channels_vs_oracle(n, dtype, rule, precision):
    rng = np.random.default_rng(50 + n)
    gates = wc.random_gate_list(n, 40, rng, max_k=2)
    lib, spots, u = _ops(n, len(gates), rng)
    st = sv.State(n, dtype)
    got = st.run_trajectory(to_binding(gates), lib, u, max_k=-1 if rule == sv.RULE_AUTO else 4, rule=rule,
                            precision=precision)
    want_psi, want = dm.trajectory(n, gates, spots, u)
    assert [int(x) for x in got] == [int(x) for x in want]
    # complex64: some 70 fused passes at most, each rounding to 2^-24 of the norm
    tol = 1e-12 if dtype == "c128" else 70 * 2.0 ** -24
    assert np.linalg.norm(st.read() - want_psi) <= tol


@pytest.mark.parametrize("n,k,dtype", [(3, 3, "c64"), (9, 9, "c128"), (13, 13, "c64"), (20, 12, "c64"), (19, 19, "c128")])
def test_measurement_of_many_qubits(n, k, dtype):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if dtype == "c64" else np.complex128)
    st = sv.State(n, dtype).write(psi)
    qs, u = [int(q) for q in rng.permutation(n)[:k]], rng.random(k)
    bits, p = st.measure(qs, u)
    want, wbits, wp = oracle_ops.measure(psi.astype(np.complex128), qs, u)
    assert bits == wbits
    assert abs(p - wp) <= 1e-12 * wp
    assert np.linalg.norm(st.read() - want) <= (1e-12 if dtype == "c128" else 8 * 2.0 ** -24)
