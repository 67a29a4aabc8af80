"""The tiled Pauli kernels (states of at least 19 qubits) against plain
complex128 sums: below their smallest state, at it, with a window that is cut
short and with two whole windows; groups of one and of many terms, real and
imaginary, inside a tile and across tiles."""
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


def _terms(n, rng):
    terms = [(0.5, ()), (-0.25, ((0, "Y"),)), (0.75, ((n - 1, "Y"), (0, "X")))]
    terms += [(float(rng.normal()), ((i, "Z"), (i + 1, "Z"))) for i in range(n - 1)]
    terms += [(float(rng.normal()), ((i, "X"),)) for i in range(n)]
    for _ in range(12):
        qs = rng.choice(n, size=int(rng.integers(1, 6)), replace=False)
        terms.append((float(rng.normal()), tuple((int(q), "XYZ"[int(rng.integers(3))]) for q in qs)))
    # many terms on one x mask, real and imaginary weights
    for q in range(2, n - 1):
        terms.append((float(rng.normal()), ((1, "X"), (q, "Z"))))
        terms.append((float(rng.normal()), ((1, "Y"), (n - 1, "X"), (q, "Z"))))
    return [t for t in terms if len({q for q, _ in t[1]}) == len(t[1])]


@pytest.mark.parametrize("n", [18, 19, 20, 21])
@pytest.mark.parametrize("dtype", ["c64", "c128"])
def test_pauli_sums_against_plain_sums(n, dtype):
    rng = np.random.default_rng(100 + n)
    psi = rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)
    psi = (psi / np.linalg.norm(psi)).astype(np.complex64 if dtype == "c64" else np.complex128)
    a, out = sv.State(n, dtype).write(psi), sv.State(n, dtype)
    psi = psi.astype(np.complex128)
    terms = _terms(n, rng)
    want = sum(c * ref.pauli_apply(psi, f) for c, f in terms)
    size = sum(abs(c) for c, _ in terms)
    # FP64 sums of the terms' products, then (H psi) one rounding to the type
    sums = len(terms) * 2.0 ** -52 * size
    assert abs(a.expectation(terms) - np.vdot(psi, want).real) <= 2 * sums
    a.apply_pauli_sum(terms, out)
    got = out.read().astype(np.complex128)
    rounding = 2.0 ** -24 if dtype == "c64" else 0.0
    for part in (np.real, np.imag):
        slack = rounding * np.abs(part(want)) + sums * np.abs(psi).max()
        assert np.all(np.abs(part(got) - part(want)) <= slack)
