"""Plans kept while the tile shape changes: passes of more positions than the
shape that is set when the plan is applied holds, against the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_FP16: 2.0 ** -20}


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()
    sv.set_tile_shape(14, 16)


@pytest.mark.parametrize("rule,max_k", [(sv.RULE_ENHANCED, 5), (sv.RULE_PAPER, 4), (sv.RULE_TILED, 4)])
@pytest.mark.parametrize("precision", list(STEP))
def test_plan_kept_over_a_new_shape(rule, max_k, precision):
    n = 16
    gates = []
    for layer in range(6):  # pairs on positions 0..13: a pass of a whole 14-bit tile
        gates += [wc.Gate("SQRT_W", (q,)) for q in range(n)]
        gates += [wc.Gate("FSIM", (q, q + 1), (1.1, 0.3)) for q in range(layer % 2, n - 1, 2)]
    bound, want, tol = to_binding(gates), ref.simulate(n, gates, "0"), len(gates) * STEP[precision]
    plan = sv.fuse(bound, n, max_k, rule, precision=precision)
    tiles = plan if rule == sv.RULE_TILED else sv.fuse(bound, n, 4, sv.RULE_TILED, precision=precision)
    unions = {}
    for b in tiles.blocks(False):
        unions.setdefault(b.tile_pass, set()).update(b.qubits)
    assert max(len(u) for p, u in unions.items() if p >= 0) == 14
    for shape in sv.TILE_SHAPES:
        sv.set_tile_shape(*shape)
        st = sv.State(n, "c64").apply_plan(plan, precision=precision)
        assert np.linalg.norm(st.read() - want) <= tol, shape
