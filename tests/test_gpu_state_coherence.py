"""States of several pieces and energies in a process whose pinned memory is not coherent
unless asked for (the HIP runtime's HIP_HOST_COHERENT=0): what goes in comes out."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = """
import numpy as np
import lion_inputs as li
from paper_1907_10514_amd import Simulation

rng = np.random.default_rng(1)
for n in (100, 50001):
    sim = Simulation(np.full(n, li.REF_MASS), np.zeros(n), "fp64", autotuned=False)
    for _ in range(20):
        rows = rng.normal(0, 1e-4, (6, n))
        sim.set_state(*rows, 0.0)
        got, _ = sim.get_state()
        for c, r in zip(("x", "y", "z", "vx", "vy", "vz"), rows):
            assert np.array_equal(got[c], r), (n, c)
        kinetic = 0.5 * li.REF_MASS * np.sum(rows[3:] ** 2)
        assert abs(sim.energy()[0] - kinetic) <= 1e-12 * kinetic
    sim.close()
print("whole")
"""


def test_not_coherent_by_default():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=ROOT, capture_output=True, text=True,
                       timeout=100, env={**os.environ, "HIP_HOST_COHERENT": "0"})
    assert r.returncode == 0 and r.stdout.strip().endswith("whole"), r.stdout + r.stderr
