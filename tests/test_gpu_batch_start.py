"""Batches whose states start in their first pass: trajectories without a gate,
of one pass and of several, below and above the LDS size, run again and again
over what the last run left, in every precision against the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20,
        sv.PREC_SPLIT_BF16: 2.0 ** -15}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()


def _gates(n, layers, rng):
    out = []
    for layer in range(layers):
        out += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(n)]
        out += [wc.Gate("FSIM", (q, (q + 7) % n), (1.1, 0.3)) for q in range(layer % 2, n, 2)]
    return out


@pytest.mark.parametrize("precision", list(STEP))
def test_states_start_in_their_first_pass(precision):
    rng = np.random.default_rng(3)
    circuits = [(n, _gates(n, layers, rng)) for n, layers in
                [(1, 0), (3, 2), (12, 5), (13, 3), (14, 0), (14, 4), (15, 1), (17, 6), (18, 0), (18, 3)]]
    batch = sv.Batch([(n, to_binding(g)) for n, g in circuits], max_k=4, precision=precision)
    want = [ref.simulate(n, g, "0") for n, g in circuits]
    first = None
    for use_graph in (False, True, True):
        z = batch.run(use_graph=use_graph)
        first = z if first is None else first
        assert np.array_equal(z, first)
        for t, ((n, g), w) in enumerate(zip(circuits, want)):
            tol = max(1, len(g)) * STEP[precision]
            assert np.linalg.norm(batch.read(t) - w) <= tol, t
            p = np.abs(w) ** 2
            assert abs(z[t] - (p[0::2].sum() - p[1::2].sum())) <= 2 * tol, t
