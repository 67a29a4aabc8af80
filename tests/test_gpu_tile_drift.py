"""FP32 and split-BF16X3 tile passes round without a bias: the trace of a noisy
density matrix, a sum of positive entries, stays at 1 over some 100 blocks."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


@pytest.mark.parametrize("n", [6, 9])
@pytest.mark.parametrize("precision", [sv.PREC_FP32, sv.PREC_SPLIT_BF16X3])
def test_trace(n, precision):
    rng = np.random.default_rng(n)
    gates, ops = [], []
    for layer in range(12):
        gates += [(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,), ()) for q in range(n)]
        for q in range(layer % 2, n - 1, 2):
            gates.append(("FSIM", (q, q + 1), (np.pi / 2, np.pi / 6)))
            ops.append(sv.depolarizing((q, q + 1), 0.01, after=len(gates)))
    rho = sv.DensityMatrix(n, "c64").run(gates, ops, max_k=4, rule=sv.RULE_TILED, precision=precision)
    # some 100 independent roundings of at most 2^-24 of each of 2^n like entries,
    # three standard deviations, and twice that for uneven entries
    assert abs(rho.trace() - 1.0) <= 2 * 3 * 10 * 2.0 ** -24 / np.sqrt(1 << n)
