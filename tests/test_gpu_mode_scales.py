"""Mode frequencies over the range of a double: couplings whose squares underflow inside an
ordinary matrix, matrices whose entries' squares overflow or underflow, with and without
the column-per-launch part of the solver (order above 192), against the oracle's dense
eigenvalues; and a Hessian that is not finite is refused on every path."""
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


def _check(oracle_mod, pos, trap):
    from paper_1907_10514_amd import Simulation

    n = pos.shape[1]
    V0, U0 = oracle_mod.voltages_for(0.25, -0.001, li.REF_MASS, li.E_CHARGE, li.OMEGA, li.R0,
                                     li.Z0, li.KAPPA) if trap else (0.0, 0.0)
    tr = oracle_mod.Trap(V0=V0, Omega=li.OMEGA, U0=U0, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA,
                         pseudo=True)
    mass, charge = np.full(n, li.REF_MASS), np.full(n, li.E_CHARGE)
    sim = Simulation(mass, charge, "fp64")
    sim.set_pseudo_trap(tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0, tr.kappa)
    sim.set_state(*pos, *np.zeros((3, n)), 0.0)
    got, _ = sim.normal_modes()
    sim.close()
    ref = np.linalg.eigvalsh(oracle_mod.hessian(*pos, charge, mass, tr))
    assert np.all(np.diff(got) >= 0)
    # entries off by a few roundings and a backward-stable reduction, of the largest
    tol = (4 * 3 * n + 60) * 2.0 ** -53 * np.max(np.abs(ref))
    assert np.max(np.abs(got - ref)) <= tol


@pytest.mark.parametrize("exponent", [-140, -155, *range(-180, -159), -300])
@pytest.mark.parametrize("n", [2, 20, 70])
def test_tiny_couplings(torch_gpu, oracle_mod, n, exponent):
    """An axial chain whose first ion is off its axis by 10^exponent m."""
    pos = np.zeros((3, n))
    pos[0, 0] = 10.0 ** exponent
    pos[2] = 7e-6 * (np.arange(n) - 0.5 * (n - 1))
    _check(oracle_mod, pos, True)


@pytest.mark.parametrize("distance", [1e48, 1e50, 1e51, 1e52, 1e53, 1e54, 1e58])
@pytest.mark.parametrize("n", [2, 3, 66, 70])
def test_far_ions(torch_gpu, oracle_mod, n, distance):
    """The first and the last ion so far out that their couplings' squares vanish."""
    pos = np.random.default_rng(n).normal(0, 1e-5 * n ** (1 / 3), (3, n))
    pos[:, 0] = distance * np.array([0.3, 0.5, 0.8])
    pos[:, -1] = -distance
    _check(oracle_mod, pos, True)


@pytest.mark.parametrize("spacing", [1e-58, 1e-52, 1e-40, 1e20, 1e40, 1e60])
@pytest.mark.parametrize("n", [1, 2, 5, 66])
def test_all_entries_large_or_small(torch_gpu, oracle_mod, n, spacing):
    """No trap: the entries go as spacing^-3."""
    pos = spacing * np.random.default_rng(n).normal(0, n ** (1 / 3), (3, n))
    _check(oracle_mod, pos, False)


@pytest.mark.parametrize("vectors", [False, True])
@pytest.mark.parametrize("n", [3, 66, 171])
def test_not_finite(torch_gpu, n, vectors):
    from paper_1907_10514_amd import LionError, Simulation
    from paper_1907_10514_amd import lion as L

    sim = Simulation(np.full(n, li.REF_MASS), np.full(n, li.E_CHARGE), "fp64")
    pos = np.random.default_rng(n).normal(0, 1e160, (3, n))  # r^2 overflows
    sim.set_state(*pos, *np.zeros((3, n)), 0.0)
    for _ in range(2):
        with pytest.raises(LionError) as ei:
            sim.normal_modes(vectors=vectors)
        assert ei.value.code == L.LION_ERR_HIP and "not finite" in str(ei.value)
    pos = np.random.default_rng(n).normal(0, 1e-5 * n ** (1 / 3), (3, n))
    sim.set_state(*pos, *np.zeros((3, n)), 0.0)  # the handle goes on
    assert np.all(np.isfinite(sim.normal_modes(vectors=vectors)[0]))
    sim.close()
