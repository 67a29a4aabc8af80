"""Set tile shapes other than the default: states of 10 to 13 qubits, whose
passes take smaller shapes with block limits of their own, against the oracle."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_SPLIT_BF16X3: 2.0 ** -21, sv.PREC_FP64: 2.0 ** -49}


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()
    sv.set_tile_shape(14, 16)


def _layers(n, count, rng):
    """Nearest-neighbour layers: passes of as many blocks as the shape holds."""
    out = []
    for layer in range(count):
        out += [wc.Gate(("SQRT_X", "SQRT_Y", "SQRT_W")[int(rng.integers(3))], (q,)) for q in range(n)]
        out += [wc.Gate("FSIM", (q, q + 1), (1.1, 0.3)) for q in range(layer % 2, n - 1, 2)]
    return out


@pytest.mark.parametrize("shape", sv.TILE_SHAPES)
@pytest.mark.parametrize("precision", list(STEP))
@pytest.mark.parametrize("n", [10, 11, 12, 13])
def test_small_states(shape, precision, n):
    gates = _layers(n, 16, np.random.default_rng(n))
    bound, dtype, tol = to_binding(gates), "c128" if precision == sv.PREC_FP64 else "c64", len(gates) * STEP[precision]
    want = ref.simulate(n, gates, "0")
    sv.set_tile_shape(*shape)
    plan = sv.fuse(bound, n, 4, sv.RULE_TILED, precision=precision)
    sizes = np.bincount([b.tile_pass for b in plan.blocks(False) if b.tile_pass >= 0])
    if shape == (13, 8) and precision != sv.PREC_FP64:
        assert max(sizes) >= 12  # more than (12, 4) holds
    for name, st in (("run", sv.State(n, dtype).run(bound, max_k=4, rule=sv.RULE_TILED, precision=precision, basis=0)),
                     ("plan", sv.State(n, dtype).apply_plan(plan, precision=precision)),
                     ("dense", sv.State(n, dtype).run(bound, max_k=5, rule=sv.RULE_ENHANCED, precision=precision)),
                     ("graph", sv.State(n, dtype).run(bound, max_k=4, rule=sv.RULE_TILED, precision=precision, use_graph=True))):
        assert np.linalg.norm(st.read() - want) <= tol, name


@pytest.mark.parametrize("n", [10, 12, 13])
def test_small_sweeps(n):
    gates = _layers(n, 16, np.random.default_rng(n))
    gates[n:n] = [wc.Gate("RY", (q,), (0.3 + q,), q) for q in range(n)]
    H = [(1.0, ((q, "Z"),)) for q in range(n)]
    grads = []
    for shape in sv.TILE_SHAPES:
        sv.set_tile_shape(*shape)
        psi = sv.State(n, "c64").run(to_binding(gates), max_k=4, rule=sv.RULE_TILED)
        grads.append(sv.backward(psi, sv.State(n, "c64"), to_binding(gates), H, n))
        # two sweeps, two states, |H| <= n
        assert np.abs(grads[-1] - grads[0]).max() <= 2 * 2 * 2 * len(gates) * STEP[sv.PREC_FP32] * n, shape
