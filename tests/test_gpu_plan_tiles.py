"""Kept plans form their tile passes when they are first applied: from copies of
the gates' matrices, once for all threads."""
import gc
import threading
import time

import numpy as np
import pytest

import paper_2111_06868_amd as sv
from helpers import to_binding
from oracle import ref
from workloads import circuits as wc

# l2 error of one block on a norm-1 state
STEP = {sv.PREC_FP32: 2.0 ** -21, sv.PREC_FP64: 2.0 ** -49}


def _gates(n, layers):
    gates = []
    for layer in range(layers):
        gates += [wc.Gate("MATRIX", (q,), (q + layer,)) for q in range(n)]
        gates += [wc.Gate("FSIM", (q, q + 1), (1.1, 0.3)) for q in range(layer % 2, n - 1, 2)]
    return gates


@pytest.mark.gpu
@pytest.mark.parametrize("precision", list(STEP))
def test_applied_after_the_gates_are_gone_by_several_threads(precision):
    import torch
    assert torch.cuda.is_available(), "GPU tests need an MI355X"
    n, gates = 15, _gates(15, 4)
    array = sv.GateArray(to_binding(gates))
    plan = sv.fuse(array, n, 5, sv.RULE_ENHANCED, precision=precision)
    for m in array._keep:
        m[:] = np.nan  # the caller's memory is its own again
    del array
    gc.collect()
    dtype = "c128" if precision == sv.PREC_FP64 else "c64"
    states = [sv.State(n, dtype).set_basis(0) for _ in range(6)]
    threads = [threading.Thread(target=st.apply_plan, args=(plan,), kwargs={"precision": precision}) for st in states]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    want = ref.simulate(n, gates, "0")
    for st in states:
        assert np.linalg.norm(st.read() - want) <= len(gates) * STEP[precision]


def test_a_plan_that_is_not_applied_does_not_form_them():
    n, array = 20, sv.GateArray(to_binding(_gates(20, 6)))

    def best(precision):
        times = []
        for _ in range(40):
            t = time.perf_counter()
            sv.fuse(array, n, 4, sv.RULE_PAPER, precision=precision)
            times.append(time.perf_counter() - t)
        return min(times)

    # split FP16 plans have none; forming them takes half as long again
    assert min(best(sv.PREC_FP32) / best(sv.PREC_SPLIT_FP16) for _ in range(3)) <= 1.25
