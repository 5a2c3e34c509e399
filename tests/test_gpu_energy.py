"""Energies of one trap and of batches at the edges of the device sum's tiles (128
targets, 256 sources), with charges of both signs, coincident ions and an ion so far
away that r^2 overflows, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu

# Plain FP64 sums of at most 128 terms inside compensated ones, each term with at most
# four roundings: 132 half-ulps of the sum of magnitudes, and as much for the oracle.
TOL = 2 * 132 * 2.0 ** -53


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def _cloud(n, seed):
    rng = np.random.default_rng(seed)
    st = dict(zip(("x", "y", "z"), rng.normal(0, 50e-6, (3, n))))
    st.update(zip(("vx", "vy", "vz"), rng.normal(0, 3.0, (3, n))))
    charge = rng.choice([-1.0, 1.0, 2.0], n) * li.E_CHARGE
    mass = rng.choice([17.0, 40.0], n) * li.AMU
    if n >= 4:
        for c in "xyz":
            st[c][n - 1] = st[c][0]  # coincident with ion 0
    return st, charge, mass


def _check(got, ref, mag):
    for g, r, m in zip(got, ref, mag):
        assert abs(g - r) <= TOL * m, (g, r, m)


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 255, 256, 257, 512, 1000, 5000])
def test_energy_of_one_trap(torch_gpu, oracle_mod, n):
    from paper_1907_10514_amd import Simulation

    st, q, m = _cloud(n, n)
    tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.24, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA)
    sim = Simulation(m, q, "fp64")
    sim.set_trap(tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0, tr.kappa)
    sim.set_state(*[st[k] for k in ("x", "y", "z", "vx", "vy", "vz")])
    ref = oracle_mod.energy(st, q, m, tr)
    mag = oracle_mod.energy(st, np.abs(q), m, tr)
    a_dc = tr.kappa * tr.U0 / tr.Z0 ** 2
    dmag = float(np.sum(np.abs(q) * a_dc * (st["x"] ** 2 + st["y"] ** 2 + st["z"] ** 2)))
    _check(sim.energy(), ref, (mag[0], mag[1], dmag))
    if n >= 4:  # r^2 to ion 1 overflows: it adds nothing to the pair sum
        far = {k: v.copy() for k, v in st.items()}
        far["x"][1] = 1e160
        sim.set_state(*[far[k] for k in ("x", "y", "z", "vx", "vy", "vz")])
        keep = np.arange(n) != 1
        ref = oracle_mod.energy({k: v[keep] for k, v in st.items()}, q[keep], m[keep], tr)
        assert abs(sim.energy()[1] - ref[1]) <= TOL * mag[1]
    sim.close()


@pytest.mark.parametrize("sizes", [[1], [300], [1, 2, 128, 129, 256, 257, 1024, 5], [20] * 400])
def test_energy_of_batches(torch_gpu, oracle_mod, sizes):
    from paper_1907_10514_amd import Simulation

    st, q, m = _cloud(sum(sizes), len(sizes))
    sim = Simulation(m, q, "fp64", n_per_trap=sizes)
    off = np.concatenate([[0], np.cumsum(sizes)])
    ref, mag = np.zeros(3), np.zeros(3)
    for k in range(len(sizes)):
        tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.1 + 0.001 * k, R0=li.R0, Z0=li.Z0,
                             kappa=li.KAPPA)
        sim.set_trap(tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0, tr.kappa, trap=k)
        sl = slice(off[k], off[k + 1])
        part = {c: v[sl] for c, v in st.items()}
        ref += oracle_mod.energy(part, q[sl], m[sl], tr)
        e = oracle_mod.energy(part, np.abs(q[sl]), m[sl], tr)
        a_dc = tr.kappa * tr.U0 / tr.Z0 ** 2
        mag += (e[0], e[1], np.sum(np.abs(q[sl]) * a_dc * sum(part[c] ** 2 for c in "xyz")))
    sim.set_state(*[st[k] for k in ("x", "y", "z", "vx", "vy", "vz")])
    _check(sim.energy(), ref, mag)
    sim.close()
