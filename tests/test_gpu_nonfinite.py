"""Infinities and NaN in the state: they stay in the cosets of the positions
that the gates act on, are never turned into numbers, and the reductions that
meet one say so, in every kernel that applies blocks or sums over the state."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state; split FP16 cannot scale by an
# infinite norm: two unscaled parts, 2^-25 for each of 2^17 real numbers
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -16, sv.PREC_SPLIT_BF16: 2.0 ** -15,
        sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_FP64: 2.0 ** -49}
BAD = [np.nan, np.inf, complex(0, -np.inf)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _state(n, dtype, at, bad):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if dtype == "c64" else np.complex128)
    psi[at] = bad
    return psi


def _coset(n, qubits, at):
    mask = sum(1 << q for q in qubits)
    return (np.arange(1 << n) & ~mask) == (at & ~mask)


def _check(st, psi, n, gates, at, tol):
    qubits = {q for g in gates for q in g.qubits}
    inside = _coset(n, qubits, at)
    got = st.read()
    start = psi.astype(np.complex128)
    start[at] = 0
    want = ref.simulate(n, gates, psi=start)  # the coset aside, the same state
    assert np.isfinite(got[~inside]).all()
    assert np.linalg.norm(got[~inside] - want[~inside]) <= tol
    # the last gate's group of a bad amplitude is bad, whichever way it spread
    assert not np.isfinite(got[inside]).all()
    last = _coset(n, gates[-1].qubits, at)
    assert not np.isfinite(got[last]).any()


def _dense(qubits, seed):
    return wc.Gate("MATRIX", qubits, (seed,))  # no zero entries


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("precision", list(STEP))
@pytest.mark.parametrize("n,rule,max_k", [(15, sv.RULE_TILED, 4), (16, sv.RULE_ENHANCED, 5), (14, sv.RULE_NONE, 6),
                                          (12, sv.RULE_TILED, 4), (9, sv.RULE_PAPER, 6), (8, sv.RULE_NONE, 6)])
def test_blocks(n, rule, max_k, precision, bad):
    gates = [_dense((0,), 1), _dense((5, 2), 2), _dense((1, 0), 3), _dense((6, 3, 1), 4), _dense((2, 6, 0, 5), 5)]
    if rule == sv.RULE_NONE:
        gates.append(_dense((7, 1, 2), 6))
    at, dtype = 0b10110101 % (1 << n), "c128" if precision == sv.PREC_FP64 else "c64"
    psi = _state(n, dtype, at, bad)
    st = sv.State(n, dtype).write(psi).run(to_binding(gates), max_k=max_k, rule=rule, precision=precision)
    _check(st, psi, n, gates, at, len(gates) * STEP[precision])


@pytest.mark.parametrize("bad", BAD)
@pytest.mark.parametrize("n,dtype", [(6, "c64"), (11, "c128"), (19, "c64"), (20, "c128")])
def test_sums(n, dtype, bad):
    at = (1 << n) - 3
    psi = _state(n, dtype, at, bad)
    st, out = sv.State(n, dtype).write(psi), sv.State(n, dtype)
    H = [(1.0, ((0, "Z"), (n - 1, "Z"))), (0.5, ((1, "X"),)), (0.25, ((n - 1, "Y"), (0, "X"))), (0.125, ((2, "Z"),))]
    assert not np.isfinite(st.norm2()) and not np.isfinite(st.expectation(H))
    st.apply_pauli_sum(H, out)
    got = out.read()
    hit = {at, at ^ 2, at ^ ((1 << (n - 1)) | 1)}  # the x masks of H
    assert set(np.flatnonzero(~np.isfinite(got)).tolist()) == hit
    for channel in (sv.amplitude_damping(0, 0.3), sv.SuperOp((0,), left=wc.random_kraus_from_seed(7, 1, 2))):
        with pytest.raises(sv.SvValueError):
            st.run_trajectory([], [channel], [0.5])
    with pytest.raises(sv.SvValueError):
        st.measure([0, n - 1], [0.5, 0.5])
    gates = [("RY", (q,), (0.3,), q) for q in range(n)]
    assert not np.isfinite(sv.backward(sv.State(n, dtype).write(psi), out, gates, H, n)).any()
