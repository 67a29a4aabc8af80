"""A trajectory of many wide channels holds the matrices of a few at a time."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SCRIPT = """
import resource
import numpy as np
import torch
assert torch.cuda.is_available()
import paper_2111_06868_amd as sv
op = sv.depolarizing((0, 1, 2), 0.3)
st = sv.State(3, "c128")
peak = lambda: resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
def run(count):
    picks = st.run_trajectory([("H", (0,))], [op.at(1) for _ in range(count)], np.linspace(0, 0.999, count))
    assert len(set(int(p) for p in picks)) > 10
run(40)
before = peak()
run(2000)
print("grown", peak() - before)
"""


def test_matrices_of_a_few_channels_at_a_time():
    out = subprocess.run([sys.executable, "-c", SCRIPT], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert out.returncode == 0, out.stderr
    # KiB: 2000 channels of 128 KiB would take 250 MiB
    assert int(out.stdout.split("grown")[1]) < 64 * 1024
