"""FP64 tile passes of complex128 states against the oracle: one block to more
than one launch holds, positions low and high, plans made for FP64 and for
another arithmetic (whose passes may cover 14 positions, one more than an
FP64 tile), runs from a basis state, in a graph, and two states at once (the
adjoint sweep)."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
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


def _tiles():
    return sum(sv.stats_query("tile_fp64", k)[0] for k in range(1, 17))


@pytest.mark.parametrize("n", [14, 15, 17])
@pytest.mark.parametrize("planned_for", [sv.PREC_FP64, None, sv.PREC_FP32])
def test_blocks_componentwise(n, planned_for):
    rng = np.random.default_rng(n)
    for count in (1, 2, 5, 7, 8, 15):
        psi = (rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)) * np.exp(3 * rng.normal(size=1 << n))
        gates, mats = [], []
        for i in range(count):
            q = tuple(int(x) for x in rng.choice(n if i % 3 else 10, size=4 - (i % 4 == 3), replace=False))
            D = 1 << len(q)
            m = (rng.normal(size=(D, D)) + 1j * rng.normal(size=(D, D))) * np.exp(3 * rng.normal(size=(D, D)))
            mats.append((m / np.linalg.norm(m, 2), q))
            gates.append(("MATRIX", q, (), -1, mats[-1][0]))
        st = sv.State(n, "c128").write(psi)
        plan = sv.fuse(gates, n, 4, sv.RULE_TILED, precision=planned_for)
        sv.stats_reset()
        sv.stats_enable(True)
        st.apply_plan(plan)
        st.synchronize()
        tiles = _tiles()
        sv.stats_enable(False)
        assert tiles >= 1
        want, size = psi.copy(), np.abs(psi).astype(np.complex128)
        for m, q in mats:
            ref.apply(want, m, q)
            ref.apply(size, np.abs(m).astype(np.complex128), q)
        # per block: 32 rounded products and sums of re and im on each side, and
        # a block may be the product of all the gates that it holds
        bound = 2 * 4 * count * 34 * 2.0 ** -53 * np.abs(size)
        assert np.all(np.abs(st.read() - want) <= bound + 1e-290)


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("rule", [sv.RULE_TILED, sv.RULE_AUTO])
def test_circuit_from_a_basis_state(use_graph, rule):
    n, gates = 16, wc.grid_rqc(4, 4, 6, 3)
    bound = to_binding(gates)
    st = sv.State(n, "c128").set_product("+")
    for basis in (0, 40961, 5):
        st.run(bound, max_k=4, rule=rule, use_graph=use_graph, basis=basis)
        psi = np.zeros(1 << n, dtype=np.complex128)
        psi[basis] = 1.0
        for g in gates:
            ref.apply(psi, ref.matrix_of(g), g.qubits)
        # some 20 blocks, each a product of FP64 gates: rounding of norm-1 vectors
        assert np.linalg.norm(st.read() - psi) <= 20 * 34 * 2.0 ** -53


def test_adjoint_sweep_in_fp64_tiles():
    n = 14
    gates, thetas = wc.ansatz_circuit(n, 3, seed=5)
    H = wc.ansatz_observable(n)
    bound = to_binding(gates)
    psi, scratch = sv.State(n, "c128").run(bound, max_k=4, rule=sv.RULE_TILED), sv.State(n, "c128")
    got = sv.backward(psi, scratch, bound, H, len(thetas))
    # parameter shift on a few angles, exact for rotations
    for p in (0, n + 3, 4 * n + 1, len(thetas) - 1):
        e = []
        for sgn in (1, -1):
            th = thetas.copy()
            th[p] += sgn * np.pi / 2
            e.append(ref.expectation(ref.simulate(n, wc.with_thetas(gates, th), "0"), H))
        assert abs(got[p] - 0.5 * (e[0] - e[1])) <= 1e-11
