"""FP32 tile passes (three BF16 parts of matrix and state): componentwise
error of launches whose operands are all expanded in LDS and of launches that
keep two parts compact, at every launch shape, for matrices and states whose
entries span many magnitudes."""
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
    sv.set_tile_shape(14, 16)
    torch.cuda.synchronize()


@pytest.mark.parametrize("shape,counts", [((14, 16), (1, 4, 5, 6, 7)), ((14, 8), (5, 7)), ((13, 4), (2, 3)),
                                          ((13, 8), (10, 16))])
@pytest.mark.parametrize("basis", [None, 11])
def test_componentwise_error(shape, counts, basis):
    sv.set_tile_shape(*shape)
    n = 15
    for count in counts:
        rng = np.random.default_rng(1000 * shape[0] + 10 * shape[1] + count)
        psi = (rng.normal(size=1 << n) + 1j * rng.normal(size=1 << n)) * np.exp(3 * rng.normal(size=1 << n))
        psi = psi.astype(np.complex64)
        mats, gates = [], []
        for i in range(count):
            # rotating positions (0 in some blocks, not in others) of a 10-position union
            q = tuple(sorted((3 * i + j * (2 + i % 2)) % 10 for j in range(4)))
            if len(set(q)) < 4:
                q = (0, 3, 6, 9)
            m = (rng.normal(size=(16, 16)) + 1j * rng.normal(size=(16, 16))) * np.exp(3 * rng.normal(size=(16, 16)))
            mats.append((m / np.linalg.norm(m, 2), q))
            gates.append(("MATRIX", q, (), -1, mats[-1][0]))
        st = sv.State(n, "c64").write(psi)
        st.run(gates, max_k=4, rule=sv.RULE_TILED, precision=sv.PREC_FP32, basis=basis)
        want = psi.astype(np.complex128)
        if basis is not None:
            want = np.zeros(1 << n, dtype=np.complex128)
            want[basis] = 1.0
        size = np.abs(want).astype(np.complex128)  # |U_s| .. |U_1| |psi|
        for m, q in mats:
            ref.apply(want, m, q)
            ref.apply(size, np.abs(m).astype(np.complex128), q)
        # per block: the parts' dropped products (below 2^-25) and the FP32
        # roundings of a sum of 12 products of 16 terms, on re and im
        bound = 2 * count * 13 * 2.0 ** -24 * np.abs(size)
        assert np.all(np.abs(st.read() - want) <= bound + 1e-37)
