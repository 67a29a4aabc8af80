"""Host planning: block matrices against numpy products of the members, and the
operand array of many super operators against SuperOp.fill (CPU)."""
import ctypes

import numpy as np
import pytest

import paper_2111_06868_amd as sv
from paper_2111_06868_amd import _native as N
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc


def _gates(n, count, rng):
    """One-qubit gates held back alone, in pairs and at the end; named and
    matrix gates of one to three qubits."""
    out = []
    for _ in range(count):
        kind = int(rng.integers(5))
        if kind < 2:
            name = ("RX", "RY", "RZ", "SQRT_W", "H")[int(rng.integers(5))]
            out.append(wc.Gate(name, (int(rng.integers(n)),), (float(rng.uniform(0, 6)),) if name[0] == "R" else ()))
        elif kind < 4:
            q = tuple(int(x) for x in rng.choice(n, 2, replace=False))
            out.append(wc.Gate(*[("CX", q), ("CZ", q), ("FSIM", q, (0.7, 0.3))][int(rng.integers(3))]))
        else:
            k = int(rng.integers(1, 4))
            out.append(wc.Gate("MATRIX", tuple(int(x) for x in rng.choice(n, k, replace=False)), (int(rng.integers(99)),)))
    return out


@pytest.mark.parametrize("max_k", [3, 4, 5, 6])
@pytest.mark.parametrize("rule", [sv.RULE_PAPER, sv.RULE_ENHANCED, sv.RULE_TILED])
def test_block_matrices(max_k, rule):
    rng = np.random.default_rng(max_k)
    gates = _gates(7, 60, rng)
    for b in sv.fuse(to_binding(gates), 7, max_k, rule).blocks():
        k, pos = len(b.qubits), {q: len(b.qubits) - 1 - j for j, q in enumerate(b.qubits)}
        local = [wc.Gate(gates[i].name, tuple(pos[q] for q in gates[i].qubits), gates[i].params)
                 for i in b.members]
        want = np.stack([ref.simulate(k, local, psi=np.eye(1 << k, dtype=complex)[c].copy()) for c in range(1 << k)], axis=1)
        # at most 60 gates of at most 8 products of unit-norm rows an entry
        assert np.abs(b.matrix - want).max() <= 60 * 8 * 2.0 ** -52


def test_super_op_array():
    rng = np.random.default_rng(0)
    m = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)
    ops = [sv.SuperOp((3,), left=m(2, 2, 2), after=0), sv.SuperOp((1, 4), left=m(3, 4, 4), right=m(2, 4, 4), s=m(3, 2), after=2),
           sv.SuperOp((0, 5, 2), superop=m(64, 64), after=7), sv.depolarizing((2, 0), 0.1, after=9).at(11)]
    for extra in ([], [sv.SuperOp((2,), left=m(1, 2, 2))]):
        if extra:
            extra[0].right = m(2, 2, 2)[:1]
            extra[0].left = np.asfortranarray(m(1, 2, 4))[:, :, :2].copy()
        got = sv._super_op_array(ops + extra)
        for i, op in enumerate(ops + extra):
            want, keep = N.sv_super_op(), []
            op.fill(want, keep)
            assert bytes(got[i]) == bytes(want)
    assert ctypes.sizeof(sv._super_op_array([])) == ctypes.sizeof(N.sv_super_op)
    with pytest.raises(ValueError):
        sv._super_op_array([sv.SuperOp((0, 1, 2, 3), left=np.eye(16))])
