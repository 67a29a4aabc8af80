"""Gate passes (runs of gates of at most 3 qubits applied in LDS tiles)
against the oracle and against the same gates applied one call at a time:
every pair and triple of a stage's row bits, gates on position 0 and on the
top positions, runs broken by wider gates, graphs, and the launch counts."""
import itertools

import numpy as np
import pytest

import paper_2111_06868_amd as sv
from oracle import ref
from workloads import circuits as wc
from helpers import to_binding

pytestmark = pytest.mark.gpu

EPS = {"c64": 2.0 ** -24, "c128": 2.0 ** -53}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _unitary(rng, k):
    d = 1 << k
    q, _ = np.linalg.qr(rng.normal(size=(d, d)) + 1j * rng.normal(size=(d, d)))
    return q


def _check(n, dtype, gates, **kw):
    rng = np.random.default_rng(9)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if dtype == "c64" else np.complex128)
    st = sv.State(n, dtype).write(psi)
    st.run([("MATRIX", q, (), -1, m) for m, q in gates], **kw)
    want = psi.astype(np.complex128)
    for m, q in gates:
        ref.apply(want, m, q)
    # a gate rounds each amplitude's sum of at most 16 products, and its matrix
    assert np.linalg.norm(st.read() - want) <= len(gates) * 18 * EPS[dtype]
    return st


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("low", [0, 1, 10])
def test_every_row_pattern(dtype, low):
    """All ordered qubit choices of 1, 2 and 3 of 4 neighbouring positions."""
    rng = np.random.default_rng(low)
    gates = []
    for k in (1, 2, 3):
        for q in itertools.permutations(range(low, low + 4), k):
            gates.append((_unitary(rng, k), q))
    _check(14, dtype, gates)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [14, 15, 18])
@pytest.mark.parametrize("rule,max_k,widest", [(sv.RULE_NONE, 6, 3), (sv.RULE_NONE, 6, 4), (sv.RULE_PAPER, 2, 2),
                                               (sv.RULE_ENHANCED, 3, 3)])
def test_random_gates(dtype, n, rule, max_k, widest):
    rng = np.random.default_rng(7 * n + max_k)
    gates = []
    for _ in range(60):
        k = int(rng.integers(1, widest + 1)) if rng.random() < 0.3 else int(rng.integers(1, min(widest, 2) + 1))
        gates.append((_unitary(rng, k), tuple(int(x) for x in rng.choice(n, size=k, replace=False))))
    for use_graph in (False, True):
        _check(n, dtype, gates, rule=rule, max_k=max_k, use_graph=use_graph)


@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_counts_and_single_calls(dtype):
    n, gates = 15, wc.grid_rqc(3, 5, 4, 2)
    bound = to_binding(gates)
    sv.stats_reset()
    sv.stats_enable(True)
    st = sv.State(n, dtype).run(bound)
    st.synchronize()
    counts = [sv.stats_query("reg", k)[0] for k in (1, 2, 3)]
    sv.stats_enable(False)
    sv.stats_reset()
    assert counts == [sum(len(g.qubits) == k for g in gates) for k in (1, 2, 3)]
    one = sv.State(n, dtype)
    for g in bound:
        one.apply_gate(g)
    # the same gates in the same order on every qubit: roundings may differ
    # only where gates on other qubits come between
    assert np.linalg.norm(st.read() - one.read()) <= len(gates) * 18 * EPS[dtype]
