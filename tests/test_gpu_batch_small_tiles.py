"""Batches whose tiles differ in magnitude: three top qubits turned by small
angles, each behind the layers before it, so that no pass holds two of them and
the tiles of a pass are 2^0, 2^-10, 2^-20 and 2^-30 of the norm.  Each eighth of
the state keeps its own relative accuracy (FP16 scales by the tile), against the
oracle."""
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


# l2 error of one block on a norm-1 state, where the values of a tile lie within
# 2^-10 of its largest (FP16: the second part's last bit is then 2^-22 of them)
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20}


def _gates(n, rng):
    gates = []
    for top in (n - 1, n - 2, n - 3):
        gates += [wc.Gate("CZ", (0, top)), wc.Gate("RY", (top,), (2 * np.arcsin(2.0 ** -10),))]
        for layer in range(12):
            gates += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(n - 3)]
            gates += [wc.Gate("FSIM", (q, q + 1), (1.1, 0.3)) for q in range(layer % 2, n - 4, 2)]
    return gates


@pytest.mark.parametrize("precision", list(STEP))
@pytest.mark.parametrize("n", [18, 20])
def test_tiles_of_different_magnitude(n, precision):
    gates = _gates(n, np.random.default_rng(n))
    bound = to_binding(gates)
    blocks = sv.fuse(bound, n, 4, sv.RULE_TILED, precision=precision).blocks(False)
    tops = {}
    for b in blocks:
        tops.setdefault(b.tile_pass, set()).update(q for q in b.qubits if q >= n - 3)
    assert max(len(t) for t in tops.values()) == 1
    batch = sv.Batch([(n, bound)], max_k=4, precision=precision)
    batch.run()
    got = batch.read(0).astype(np.complex128).reshape(8, -1)
    want = ref.simulate(n, gates, "0").reshape(8, -1)
    for h in range(8):
        err, size = np.linalg.norm(got[h] - want[h]), np.linalg.norm(want[h])
        print("eighth %d: norm %.2e, relative error %.2e" % (h, size, err / size))
        assert err <= len(blocks) * STEP[precision] * size
