"""Tile passes of states of one or few tiles (10 to 13 qubits in FP32 and FP64,
every one below and above them too) against the oracle: every rule, whole-state
unions, from a basis state, captured, and in the two-state sweep."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20,
        sv.PREC_SPLIT_BF16: 2.0 ** -15, sv.PREC_FP64: 2.0 ** -49}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _gates(n, rng):
    out = []
    for layer in range(4):
        out += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(n)]
        out += [wc.Gate("FSIM", (q, (q + 1 + 2 * layer) % n), (1.1, 0.3)) for q in range(layer % 2, n, 2)
                if (q + 1 + 2 * layer) % n != q]
        out.append(wc.Gate("MATRIX", tuple(int(q) for q in rng.choice(n, 4, replace=False)), (layer,)))
    return out


@pytest.mark.parametrize("n", [9, 10, 11, 12, 13])
@pytest.mark.parametrize("precision", list(STEP))
def test_against_oracle(n, precision):
    gates = _gates(n, np.random.default_rng(n))
    bound, dtype, tol = to_binding(gates), "c128" if precision == sv.PREC_FP64 else "c64", len(gates) * STEP[precision]
    for b in (0, (1 << n) - 2):
        start = np.zeros(1 << n, complex)
        start[b] = 1.0
        want = ref.simulate(n, gates, psi=start)
        for rule, k in ((sv.RULE_TILED, 4), (sv.RULE_ENHANCED, 4), (sv.RULE_PAPER, 5), (sv.RULE_AUTO, -1)):
            st = sv.State(n, dtype).set_product("+")
            st.run(bound, max_k=k, rule=rule, precision=precision, basis=b)
            assert np.linalg.norm(st.read() - want) <= tol, (b, rule)
            st.set_basis(b).run(bound, max_k=k, rule=rule, precision=precision, use_graph=True)
            assert np.linalg.norm(st.read() - want) <= tol, (b, rule, "graph")
            plan = sv.fuse(bound, n, k, rule, precision=precision)
            st.set_basis(b).apply_plan(plan, precision=precision)
            assert np.linalg.norm(st.read() - want) <= tol, (b, rule, "plan")


@pytest.mark.parametrize("n", [10, 11, 12, 13])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_sweep(n, dtype):
    gates = _gates(n, np.random.default_rng(n))
    gates[n:n] = [wc.Gate("RY", (q,), (0.3 + q,), q) for q in range(n)]
    H = [(1.0, ((q, "Z"),)) for q in range(n)]
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    psi.run(to_binding(gates), max_k=4, rule=sv.RULE_TILED)
    got = sv.backward(psi, lam, to_binding(gates), H, n)
    step = STEP[sv.PREC_FP64 if dtype == "c128" else sv.PREC_FP32]
    for q in (0, n // 2, n - 1):
        e = []
        for s in (1, -1):
            shifted = list(gates)
            shifted[n + q] = wc.Gate("RY", (q,), (0.3 + q + s * np.pi / 2,), q)
            e.append(ref.expectation(ref.simulate(n, shifted, "0"), H))
        assert abs(got[q] - 0.5 * (e[0] - e[1])) <= 2 * 2 * len(gates) * step * n  # two sweeps, two states, |H| <= n
