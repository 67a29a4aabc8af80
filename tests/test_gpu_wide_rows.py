"""Dense blocks one output a thread on a state of 2^32 amplitudes, more than a
launch has work-items: every amplitude of a product state."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [5, 6])
def test_32_qubits(k):
    import torch
    n, D = 32, 1 << k
    rng = np.random.default_rng(k)
    U = np.linalg.qr(rng.normal(size=(D, D)) + 1j * rng.normal(size=(D, D)))[0]
    qubits = (31, 30, 0, 17, 5, 12)[:k]  # the first is the most significant bit of the local index
    st = sv.State(n, "c128").set_product("+")
    st.apply_gate(("MATRIX", qubits, (), -1, U))
    rows = U.sum(axis=1) * 2.0 ** -16
    count = 1 << 18
    for first in (0, 5 << 28, 11 << 28, (1 << 32) - count):
        i = np.arange(first, first + count, dtype=np.uint64)
        local = np.zeros(count, np.int64)
        for q in qubits:
            local = 2 * local + ((i >> np.uint64(q)) & np.uint64(1)).astype(np.int64)
        # sums of at most 64 terms of at most 2^-16 each
        assert np.abs(st.read(first, count) - rows[local]).max() <= 64 * 2.0 ** -16 * 64 * 2.0 ** -53, first
    assert abs(st.norm2() - 1) <= 1e-12
    st.free()
    torch.cuda.empty_cache()
