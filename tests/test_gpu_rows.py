"""Dense blocks of three to six qubits, one output a thread, against the oracle:
states of one group and fewer amplitudes than a workgroup up to many
workgroups, low, high and spread positions, one state and two."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("k", [3, 4, 5, 6])
@pytest.mark.parametrize("n", [3, 4, 5, 6, 7, 8, 9, 13, 14, 17])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_blocks(n, k, dtype):
    if k > n:
        pytest.skip("block wider than the state")
    rng = np.random.default_rng(100 * n + k)
    start = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    start /= np.linalg.norm(start)
    for pos in (range(k), range(n - k, n), rng.permutation(n)[:k]):
        gates = [wc.Gate("MATRIX", tuple(int(p) for p in pos), (k,))]
        st = sv.State(n, dtype)
        st.write(start)
        st.run(to_binding(gates), max_k=k, rule=sv.RULE_NONE)
        # 2^k products of rows of norm 1, twice for the input's rounding
        step = (2.0 ** -52 if dtype == "c128" else 2.0 ** -23) * 2 * (1 << k)
        assert np.linalg.norm(st.read() - ref.simulate(n, gates, psi=start.copy())) <= step


@pytest.mark.parametrize("n", [5, 8])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_two_states(n, dtype):
    """The sweep's dagger blocks act on both states in one launch."""
    gates = [wc.Gate("RY", (q,), (0.3 + q,), q) for q in range(n)]
    gates += [wc.Gate("MATRIX", tuple(range(5)), (3,)), wc.Gate("MATRIX", (4, 1, 0, 2), (5,))]
    H = [(1.0, ((0, "Z"), (n - 1, "X")))]
    psi, lam = sv.State(n, dtype), sv.State(n, dtype)
    psi.run(to_binding(gates), max_k=5, rule=sv.RULE_PAPER)
    got = sv.backward(psi, lam, to_binding(gates), H, n)
    for q in (0, n - 1):
        e = []
        for s in (1, -1):
            shifted = list(gates)
            shifted[q] = wc.Gate("RY", (q,), (0.3 + q + s * np.pi / 2,), q)
            e.append(ref.expectation(ref.simulate(n, shifted, "0"), H))
        # 2 x some ten blocks of 32 products each
        assert abs(got[q] - 0.5 * (e[0] - e[1])) <= 20 * 64 * (2.0 ** -52 if dtype == "c128" else 2.0 ** -23)
