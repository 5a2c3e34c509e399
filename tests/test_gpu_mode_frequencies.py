"""Mode frequencies alone (no vectors) at the edges of their solver's paths (order 64, 128
and 192 inside one workgroup, a column per launch above, the library above 512) against
the oracle's dense eigenvalues, with neutral ions (zero rows, repeated eigenvalues)."""
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


@pytest.mark.parametrize("neutral", [0.0, 0.4, 1.0])
@pytest.mark.parametrize("n", [1, 2, 3, 21, 22, 42, 43, 64, 65, 66, 128, 170, 171])
def test_frequencies_match_oracle(torch_gpu, oracle_mod, n, neutral):
    from paper_1907_10514_amd import Simulation

    rng = np.random.default_rng(n)
    s = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij")).reshape(3, -1)[:, :n]
    pos = 12e-6 * (g - 0.5 * (s - 1) + rng.uniform(-0.2, 0.2, (3, n)))
    mass = rng.choice([17.0, 40.0], n) * li.AMU
    charge = np.where(rng.random(n) < neutral, 0.0, rng.choice([1.0, 2.0], n)) * li.E_CHARGE
    V0, U0 = oracle_mod.voltages_for(0.25, -0.001, li.REF_MASS, li.E_CHARGE, li.OMEGA, li.R0,
                                     li.Z0, li.KAPPA)
    tr = oracle_mod.Trap(V0=V0, Omega=li.OMEGA, U0=U0, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA,
                         pseudo=True)
    sim = Simulation(mass, charge, "fp64")
    sim.set_pseudo_trap(tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0, tr.kappa)
    sim.set_state(*pos, *np.zeros((3, n)), 0.0)
    got, _ = sim.normal_modes()
    sim.close()
    ref = np.linalg.eigvalsh(oracle_mod.hessian(*pos, charge, mass, tr))
    assert np.all(np.diff(got) >= 0)
    # Weyl: entries off by a few roundings and a backward-stable reduction move an
    # eigenvalue by at most a small multiple of order times rounding of the largest
    tol = (4 * 3 * n + 60) * 2.0 ** -53 * np.max(np.abs(ref))
    assert np.max(np.abs(got - ref)) <= tol
