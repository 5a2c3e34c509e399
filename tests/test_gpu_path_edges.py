"""Sizes at which a single trap changes kernels or their shape: forces of the one-launch
step (1, 2 and 4 targets per workgroup, up to 4096 ions), the all-pairs and the rotating
pair-once kernel (20 to 22 tiles of 256 ions and from 26), with one common charge and with
several, and short runs of the smallest traps, against the oracle."""
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


def _sim(n, prec, uniform):
    from paper_1907_10514_amd import Simulation

    rng = np.random.default_rng(n)
    pos, vel = rng.normal(0, 10e-6 * n ** (1 / 3), (3, n)), rng.normal(0, 1.0, (3, n))
    mass = rng.choice([17.0, 40.0], n) * li.AMU
    charge = (np.ones(n) if uniform else rng.choice([-1.0, 0.0, 1.0, 2.0], n)) * li.E_CHARGE
    sim = Simulation(mass, charge, prec)
    sim.set_trap(9.0, li.OMEGA, 0.24, li.R0, li.Z0, li.KAPPA)
    sim.set_state(*pos, *vel, 0.0)
    return sim, pos, vel, mass, charge


@pytest.mark.parametrize("uniform", [True, False])
@pytest.mark.parametrize("n", [257, 1536, 1537, 4095, 4096, 4097, 4864, 4865, 5632, 5633, 6400,
                               6401, 8193])
def test_forces(torch_gpu, oracle_mod, n, uniform):
    sim, pos, _, mass, charge = _sim(n, "fp64", uniform)
    tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.24, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA)
    got = np.array(sim.compute_accel())
    sim.close()
    ref = np.array(oracle_mod.accel(*pos, charge, mass, tr, 0.0))
    scale = oracle_mod.accel_scale(*pos, charge, mass, tr, 0.0)
    assert np.all(np.sqrt(((got - ref) ** 2).sum(0)) <= 1e-12 * scale)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-5), ("mixed_kahan", 1e-5)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 16, 17, 24, 48])
def test_short_runs(torch_gpu, oracle_mod, n, prec, tol):
    sim, pos, vel, mass, charge = _sim(n, prec, True)
    sim.set_damping(1e5)
    sim.step(20, li.DT)
    got, _ = sim.get_state()
    sim.close()
    tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.24, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA)
    st = dict(zip(("x", "y", "z", "vx", "vy", "vz"), (*pos, *vel)))
    ref = oracle_mod.step(st, charge, mass, tr, 1e5, 0.0, li.DT, 20)
    for c in ("x", "y", "z", "vx", "vy", "vz"):
        assert np.max(np.abs(got[c] - ref[c])) <= tol * np.max(np.abs(ref[c])), c
