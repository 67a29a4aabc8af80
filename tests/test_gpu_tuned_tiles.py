"""The autotuner measures every tile pass that plans are priced with: FP64's and
those of states below 14 qubits too, not a default scaled by the dense block."""
import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    yield
    torch.cuda.synchronize()
    sv.set_tile_shape(14, 16)


@pytest.mark.parametrize("n,precision,measured", [(16, sv.PREC_FP64, True), (11, sv.PREC_FP64, True),
                                                  (12, sv.PREC_FP32, True), (12, sv.PREC_SPLIT_BF16X3, True),
                                                  (12, sv.PREC_SPLIT_FP16, False), (9, sv.PREC_FP64, False)])
def test_tile_costs_are_measured(n, precision, measured, tmp_path, monkeypatch):
    path = tmp_path / "tune"
    monkeypatch.setenv("SV_TUNE_CACHE", str(path))
    dtype = "c128" if precision == sv.PREC_FP64 else "c64"
    sv.autotune(sv.State(n, dtype), precision)
    values = [float(x) for x in path.read_text().split()[4:26]]  # k = 1..6, then 1..16 blocks
    dense4, tiles = values[3], np.array(values[6:22])
    scaled = dense4 / 1.02 * (0.9 + 0.07 * np.arange(1, 17))
    assert (np.abs(tiles - scaled).max() > 1e-9 * dense4) == measured
    gates = wc.random_gate_list(n, 40, np.random.default_rng(n), max_k=2)
    st = sv.State(n, dtype).run(to_binding(gates), max_k=-1, rule=sv.RULE_AUTO, precision=precision)
    # the l2 error of one block on a norm-1 state, a block a gate at most
    step = {sv.PREC_FP64: 2.0 ** -49, sv.PREC_SPLIT_FP16: 2.0 ** -20}.get(precision, 2.0 ** -21)
    assert np.linalg.norm(st.read() - ref.simulate(n, gates, "0")) <= len(gates) * step


def test_dense_costs_are_those_of_the_launched_kernel():
    """FP64 blocks of three qubits below 14 take one output a thread, like those
    of four; the register kernel, six times as slow there, is not what is timed."""
    cost = sv.autotune(sv.State(12, "c128"), sv.PREC_FP64)
    assert cost[3] <= 3 * cost[4]
