"""Minimisation at the edges of its three paths (one workgroup up to 160 ions, one launch
per iteration up to 2048 in workgroups of 1, 2, 4 and 8 ions, pair kernels above) against
the oracle: two calls in a row, the second going on from the first's velocities, and a call
that stops at once."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu

# force error of the pair paths, of the force scale (as in the parity tests)
TOL = {"fp64": 1e-12, "mixed": 1e-6, "mixed_kahan": 1e-6}
DT, DMAX = 1e-8, 1e-6


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_kahan"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 160, 161, 256, 257, 512, 513, 1023, 1025,
                               2048, 2049])
def test_minimize_matches_oracle(torch_gpu, oracle_mod, n, prec):
    from paper_1907_10514_amd import Simulation

    rng = np.random.default_rng(n)
    s = int(np.ceil(n ** (1 / 3)))
    g = np.stack(np.meshgrid(*[np.arange(s)] * 3, indexing="ij")).reshape(3, -1)[:, :n]
    pos = 12e-6 * (g - 0.5 * (s - 1) + rng.uniform(-0.2, 0.2, (3, n)))
    mass = rng.choice([17.0, 40.0], n) * li.AMU
    charge = rng.choice([1.0, 2.0], n) * li.E_CHARGE
    st = dict(zip(("x", "y", "z"), pos))
    st.update({c: np.zeros(n) for c in ("vx", "vy", "vz")})
    V0, U0 = oracle_mod.voltages_for(0.25, -0.001, li.REF_MASS, li.E_CHARGE, li.OMEGA, li.R0,
                                     li.Z0, li.KAPPA)
    tr = oracle_mod.Trap(V0=V0, Omega=li.OMEGA, U0=U0, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA,
                         pseudo=True)
    sim = Simulation(mass, charge, prec)
    sim.set_pseudo_trap(tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0, tr.kappa)
    sim.set_state(*[st[c] for c in ("x", "y", "z", "vx", "vy", "vz")], 0.0)
    scale = float(np.max(mass * oracle_mod.accel_scale(*pos, charge, mass, tr, 0.0)))
    it, fmax = sim.minimize(DT, DMAX, 10 * scale)
    assert it == 0
    got = sim.get_state()[0]
    assert all(np.array_equal(got[c], st[c]) for c in st)
    done = 0
    for iters in (5, 7):
        ref = oracle_mod.minimize(st, charge, mass, tr, dt=DT, dmax=DMAX, ftol=0.0,
                                  max_iter=iters)
        it, fmax = sim.minimize(DT, DMAX, 0.0, max_iter=iters)
        got = sim.get_state()[0]
        assert it == iters == ref["iterations"]
        done += iters
        # each move is at most DMAX and its direction off by the force error; the
        # factor 20 leaves room for its growth over the moves that follow
        tol = 20 * done * DMAX * TOL[prec]
        for c in ("x", "y", "z"):
            assert np.max(np.abs(got[c] - ref[c])) <= tol, c
            assert np.max(np.abs(got["v" + c] - ref["v" + c])) <= tol / DT, c
        assert abs(fmax - ref["fmax"]) <= 10 * TOL[prec] * scale
        st = {c: ref[c] for c in st}
    sim.close()
