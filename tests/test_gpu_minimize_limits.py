"""Minimisation in one workgroup, in one launch per iteration and with the pair kernels: the
largest max_iter ends at the force tolerance, and a call longer than a launch gives the bits
of two shorter calls."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu
DT, DMAX = 1e-8, 1e-6


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def _sim(oracle_mod, n):
    from paper_1907_10514_amd import Simulation

    s = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij")).reshape(3, -1)[:, :n]
    pos = 12e-6 * (g - 0.5 * (s - 1) + np.random.default_rng(n).uniform(-0.2, 0.2, (3, n)))
    V0, U0 = oracle_mod.voltages_for(0.25, -0.001, li.REF_MASS, li.E_CHARGE, li.OMEGA, li.R0,
                                     li.Z0, li.KAPPA)
    sim = Simulation(np.full(n, li.REF_MASS), np.full(n, li.E_CHARGE), "fp64")
    sim.set_pseudo_trap(V0, li.OMEGA, U0, li.R0, li.Z0, li.KAPPA)
    sim.set_state(*pos, *np.zeros((3, n)), 0.0)
    return sim


@pytest.mark.parametrize("n", [20, 200, 2100])
def test_largest_max_iter(torch_gpu, oracle_mod, n):
    sim = _sim(oracle_mod, n)
    _, f0 = sim.minimize(DT, DMAX, 0.0, max_iter=0)
    it, f = sim.minimize(DT, DMAX, 0.8 * f0, max_iter=2 ** 63 - 1)
    assert 0 < it < 2000 and f <= 0.8 * f0
    sim.close()


@pytest.mark.parametrize("n,parts", [(20, (2000, 2001)), (160, (1999, 2)), (200, (50, 51)),
                                     (2100, (49, 2))])
def test_long_calls(torch_gpu, oracle_mod, n, parts):
    out = []
    for calls in ((sum(parts),), parts):
        sim = _sim(oracle_mod, n)
        for k in calls:
            it, _ = sim.minimize(DT, DMAX, 0.0, max_iter=k)
            assert it == k
        out.append([*sim.get_state()[0].values()])
        sim.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
