"""Sums of few and of many Pauli terms on both sides of the rules that choose
the kernel (by the terms, their groups and the state's size), <H> and H psi,
against the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from oracle import ref

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _terms(n, count, kind, rng):
    if kind in "XYZ":
        return [(float(rng.normal()), ((int((5 * i) % n), kind),)) for i in range(count)]
    return [(float(rng.normal()), tuple((int(q), "XYZ"[int(rng.integers(3))]) for q in rng.choice(n, 4, replace=False)))
            for _ in range(count)]


@pytest.mark.parametrize("dtype", ["c64", "c128"])
@pytest.mark.parametrize("n", [18, 19, 20, 22])
def test_few_and_many_terms(n, dtype):
    rng = np.random.default_rng(n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if dtype == "c64" else np.complex128)
    st, out = sv.State(n, dtype).write(psi), sv.State(n, dtype)
    x = psi.astype(np.complex128)
    for kind in "XYZr":
        for count in (1, 2, 3, 5, 9):
            H = _terms(n, count, kind, rng)
            size = sum(abs(c) for c, _ in H)
            want = sum(c * ref.pauli_apply(x, f) for c, f in H)
            got = st.apply_pauli_sum(H, out).read()
            # FP64 sums, rounded once to the amplitudes' type
            tol = size * (2.0 ** -24 if dtype == "c64" else count * 2.0 ** -52)
            assert np.linalg.norm(got - want) <= tol, (kind, count)
            assert abs(st.expectation(H) - np.vdot(x, want).real) <= size * 1e-12, (kind, count)
