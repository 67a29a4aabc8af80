"""Tile passes at the sizes where the launch shape changes (2^12, 2^13 and 2^14
unit tiles), with unions that force the next shape: 11 to 14 positions, with
and without position 0; one state, two states (adjoint sweep), from a basis
state, against the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20, sv.PREC_SPLIT_BF16: 2.0 ** -15, sv.PREC_FP64: 2.0 ** -49}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _gates(n, width, low, seed):
    """Blocks on `width` neighbouring positions from `low` up, then on as many at the top."""
    rng, gates = np.random.default_rng(seed), []
    for pos in (range(low, low + width), range(n - width, n)):
        pos = [p for p in pos if p < n]
        gates += [wc.Gate("SQRT_W", (p,)) for p in pos]
        gates += [wc.Gate("FSIM", (a, b), (0.9, 0.4)) for a, b in zip(pos[:-1], pos[1:])]
        gates += [wc.Gate("MATRIX", tuple(int(q) for q in rng.choice(pos, 4, replace=False)), (s,)) for s in range(3)]
    return gates


@pytest.mark.parametrize("n", [14, 15, 19, 20, 21, 22])
@pytest.mark.parametrize("width,low", [(10, 0), (11, 1), (12, 0), (12, 1), (13, 1), (14, 0)])
def test_shapes(n, width, low):
    gates = _gates(n, width, low, width + low)
    want = ref.simulate(n, gates, "0")
    for precision, step in STEP.items():
        st = sv.State(n, "c128" if precision == sv.PREC_FP64 else "c64")
        st.set_product("+").run(to_binding(gates), max_k=4, rule=sv.RULE_TILED, precision=precision, basis=0)
        assert np.linalg.norm(st.read() - want) <= len(gates) * step, precision


@pytest.mark.parametrize("n,dtype", [(18, "c128"), (19, "c64"), (19, "c128"), (20, "c64"), (21, "c64")])
def test_two_states(n, dtype):
    """The sweep undoes both states in launches of two: it ends at |0..0>."""
    gates = _gates(n, 12, 1, n)
    gates[3:3] = [wc.Gate("RY", (n - 1,), (0.7,), 0), wc.Gate("RX", (1,), (0.2,), 1)]
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    psi.run(to_binding(gates), max_k=4, rule=sv.RULE_TILED)
    H = [(1.0, ((n - 1, "Z"),)), (0.5, ((1, "X"), (2, "Y")))]
    got = sv.backward(psi, lam, to_binding(gates), H, 2)
    step = STEP[sv.PREC_FP64 if dtype == "c128" else sv.PREC_FP32]
    for p, i in ((0, 3), (1, 4)):
        e = []
        for s in (1, -1):
            shifted = list(gates)
            shifted[i] = wc.Gate(gates[i].name, gates[i].qubits, (gates[i].params[0] + s * np.pi / 2,), p)
            e.append(ref.expectation(ref.simulate(n, shifted, "0"), H))
        assert abs(got[p] - 0.5 * (e[0] - e[1])) <= 2 * 2 * len(gates) * step * 1.5  # both sweeps, two states, |H| <= 1.5
    back = psi.read()
    back[0] -= 1.0
    assert np.linalg.norm(back) <= 2 * len(gates) * step
