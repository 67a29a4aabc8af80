"""Planning time of tiled plans: in proportion to the number of gates (CPU)."""
import time

import paper_2111_06868_amd as sv


def _plan_time(layers):
    n, gates = 28, []
    for layer in range(layers):
        gates += [("H", (q,), ()) for q in range(n)]
        gates += [("CZ", (q, q + 1), ()) for q in range(layer % 2, n - 1, 2)]
    ga, best = sv.GateArray(gates), float("inf")
    for _ in range(3):
        t = time.perf_counter()
        sv.fuse(ga, n, 4, sv.RULE_TILED, precision=sv.PREC_SPLIT_BF16X3)
        best = min(best, time.perf_counter() - t)
    return best


def test_gates_given_back_cost_no_more_than_themselves():
    """Passes of two blocks hand most of what they took back to the planner:
    eight times the gates take eight to ten times as long, and 38 times if
    every pass looks at all gates that are left."""
    sv.set_tile_shape(13, 4)
    try:
        assert _plan_time(2000) <= 20 * _plan_time(250)
    finally:
        sv.set_tile_shape(14, 16)
