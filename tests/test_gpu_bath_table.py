"""Bath draws made ahead of the steps in blocks of half-steps: a run whose launches span
several blocks (one workgroup per trap, one launch per step, pair kernel with epilogue)
gives the bits of the same run in launches shorter than a block."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def _run(sizes, n, steps, chunk, batched, prec):
    from paper_1907_10514_amd import Simulation

    rng = np.random.default_rng(n)
    st = rng.normal(0, 10e-6 * n ** (1 / 3), (3, n)), rng.normal(0, 3.0, (3, n))
    mass = np.where(np.arange(n) % 3 == 0, 17.0, 40.0) * li.AMU
    sim = Simulation(mass, np.full(n, li.E_CHARGE), prec, n_per_trap=sizes if batched else None,
                     autotuned=False)
    sim.set_config(chunk_steps=chunk)
    sim.set_trap(9.0, li.OMEGA, 0.24, li.R0, li.Z0, li.KAPPA)
    sim.set_damping(1e4)
    sim.set_species((mass < 20 * li.AMU).astype(np.int32))
    sim.set_beam(1, (0.3, 0.2, 1.0), 2e5, species=0)
    sim.set_bath(0, 1e-3, 50e-6, 11, species=1)
    sim.set_bath(2, 2e-3, 80e-6, 12)
    sim.set_time_average(7)
    sim.set_state(*st[0], *st[1], 0.0)
    sim.step(steps, li.DT)
    out = [*sim.get_state()[0].values(), *sim.time_average()[0]]
    sim.close()
    return out


@pytest.mark.parametrize("sizes,steps,prec,batched", [
    ([16], 1100, "fp64", False),     # one wave, 512 steps per block
    ([100], 1100, "fp64", False),    # one workgroup
    ([2048], 600, "mixed", False),   # one launch per step, 511 steps per block
    ([16384], 150, "mixed", False),  # pair kernel + epilogue, 63 steps per block
    ([40] * 512, 120, "fp64", True),  # a batch, 51 steps per block
    ([700] * 30, 120, "mixed", True),
])
def test_blocks_leave_no_trace(torch_gpu, sizes, steps, prec, batched):
    n = sum(sizes)
    long = _run(sizes, n, steps, 1000, batched, prec)
    short = _run(sizes, n, steps, 13, batched, prec)
    for a, b in zip(long, short):
        assert np.all(np.isfinite(a))
        assert np.array_equal(a, b)
