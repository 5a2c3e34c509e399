"""Baths with and without memory for draws ahead of the steps: none, too little, three
half-steps, the Python layer's and far more give the same bits on every stepping path, also
when it comes or goes between calls; batches that draw in their kernels agree with the
oracle at the edges of these kernels."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6, "mixed_kahan": 1e-6}  # of the force scale
K = np.array([0.3, 0.2, 1.0]) / np.linalg.norm([0.3, 0.2, 1.0])
BEAMS = [dict(k=K, gamma=2e5, species=0)]
BATHS = [dict(temperature=1e-3, tau=50e-6, seed=11, species=1),
         dict(temperature=0.0, tau=0.0, seed=0),
         dict(temperature=2e-3, tau=80e-6, seed=12)]


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


def _table(n, half_steps):
    return 8 * ((n + 63) // 64 * 64) * (1 + 3 * half_steps)


def _setup(sim, mass, baths=True):
    sim.set_trap(9.0, li.OMEGA, 0.24, li.R0, li.Z0, li.KAPPA)
    sim.set_damping(1e4)
    sim.set_species((mass < 20 * li.AMU).astype(np.int32))
    sim.set_beam(1, (0.3, 0.2, 1.0), 2e5, species=0)
    if baths:
        sim.set_bath(0, 1e-3, 50e-6, 11, species=1)
        sim.set_bath(2, 2e-3, 80e-6, 12)
    sim.set_time_average(7)


def _inputs(n):
    rng = np.random.default_rng(n)
    mass = np.where(np.arange(n) % 3 == 0, 17.0, 40.0) * li.AMU
    return mass, [*rng.normal(0, 10e-6 * n ** (1 / 3), (3, n)), *rng.normal(0, 3.0, (3, n))]


def _run(monkeypatch, n, prec, extra, bodies=False, sizes=None):
    from paper_1907_10514_amd import Simulation
    from paper_1907_10514_amd import lion as L

    if extra is not None:
        monkeypatch.setattr(L, "bath_memory_bytes", lambda _n, _batched: extra)
    mass, rows = _inputs(n)
    sim = Simulation(mass, np.full(n, li.E_CHARGE), prec, autotuned=False,
                     n_per_trap=sizes)
    _setup(sim, mass)
    monkeypatch.undo()
    sim.set_state(*rows, 0.0)
    if bodies:  # exclusion alone, then rigid bodies: both take pair kernel and epilogue
        body = np.where(np.arange(n) < 24, np.arange(n) // 8, -1).astype(np.int32)
        sim.set_bodies(body)
        sim.step(9, li.DT)
        sim.set_rigid_bodies(body)
    out = []
    for steps in (5, 1, 60, 2):
        sim.step(steps, li.DT)
        out += [*sim.get_state()[0].values()]
    L.lion_set_bath_memory(sim.h, 0, 0)
    sim.step(6, li.DT)
    if extra:
        L.lion_set_bath_memory(sim.h, (sim._bath_memory.data_ptr() + 255) // 256 * 256, extra)
    sim.step(6, li.DT)
    out += [*sim.time_average()[0]]
    sim.set_bath(0, 0.0, 0.0, 0)
    sim.set_bath(2, 0.0, 0.0, 0)
    sim.step(8, li.DT)
    sim.set_bath(1, 1e-3, 60e-6, 5)
    sim.step(8, li.DT)
    out += [*sim.get_state()[0].values()]
    sim.close()
    return out


@pytest.mark.parametrize("n,prec,bodies", [
    (1, "fp64", False), (16, "fp64", False), (17, "mixed", False), (48, "mixed_kahan", False),
    (100, "fp64", False), (128, "mixed", False), (129, "fp64", False), (300, "mixed", False),
    (1024, "mixed_kahan", False), (2049, "mixed", False), (4097, "fp64", False),
    (5000, "fp64", False), (8192, "mixed", False), (60, "fp64", True), (700, "mixed", True)])
def test_memory_leaves_no_trace(torch_gpu, monkeypatch, n, prec, bodies):
    ref = _run(monkeypatch, n, prec, 0, bodies)
    for extra in (_table(n, 3) - 8, _table(n, 3), _table(n, 4), None, _table(n, 3000)):
        for a, b in zip(ref, _run(monkeypatch, n, prec, extra, bodies)):
            assert np.all(np.isfinite(a))
            assert np.array_equal(a, b), extra


@pytest.mark.parametrize("sizes,prec", [([16] * 9, "fp64"), ([20, 3] * 9, "mixed"),
                                        ([100, 64, 2] * 3, "mixed_kahan"),
                                        ([1024, 300, 5], "fp64")])
def test_memory_leaves_no_trace_in_batches(torch_gpu, monkeypatch, sizes, prec):
    n = sum(sizes)
    ref = _run(monkeypatch, n, prec, 0, sizes=sizes)
    for extra in (_table(n, 31), _table(n, 32), None, _table(n, 3000)):
        for a, b in zip(ref, _run(monkeypatch, n, prec, extra, sizes=sizes)):
            assert np.all(np.isfinite(a))
            assert np.array_equal(a, b), extra


def test_misaligned_memory_is_refused(torch_gpu):
    from paper_1907_10514_amd import LionError, Simulation
    from paper_1907_10514_amd import lion as L

    sim = Simulation(np.full(3, li.REF_MASS), np.full(3, li.E_CHARGE), "fp64")
    buf = torch_gpu.empty(4096, dtype=torch_gpu.uint8, device="cuda")
    with pytest.raises(LionError) as ei:
        L.lion_set_bath_memory(sim.h, (buf.data_ptr() + 255) // 256 * 256 + 8, 2048)
    assert ei.value.code == L.LION_ERR_WORKSPACE
    sim.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_kahan"])
@pytest.mark.parametrize("sizes", [[1] * 40, [2, 16, 9], [20] * 30, [1, 32, 48, 3], [49, 7],
                                   [64] * 5, [65, 200], [255, 1], [256, 30], [1024, 3, 700]])
def test_batches(torch_gpu, oracle_mod, monkeypatch, sizes, prec):
    from paper_1907_10514_amd import Simulation
    from paper_1907_10514_amd import lion as L

    n = sum(sizes)
    mass, rows = _inputs(n)
    # one trap's ions close enough to interact, none so close that rounding grows
    pos = np.concatenate([np.random.default_rng(m).normal(0, 30e-6 * m ** (1 / 3), (3, m))
                          for m in sizes], axis=1)
    monkeypatch.setattr(L, "bath_memory_bytes", lambda _n, _batched: 0)
    got = []
    for chunk in (1000, 3):
        sim = Simulation(mass, np.full(n, li.E_CHARGE), prec, n_per_trap=sizes, autotuned=False)
        sim.set_config(chunk_steps=chunk)
        _setup(sim, mass)
        sim.set_time_average(20)
        sim.set_state(*pos, *rows[3:], 0.0)
        sim.step(7, li.DT)
        sim.step(13, li.DT)
        got.append([*sim.get_state()[0].values(), *sim.time_average()[0]])
        sim.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.24, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA)
    o = 0
    for m in sizes:
        part = [a[o:o + m] for a in (*pos, *rows[3:])]
        q, w = np.full(m, li.E_CHARGE), mass[o:o + m]
        ref = oracle_mod.step_cooled(
            dict(zip(("x", "y", "z", "vx", "vy", "vz"), part)), q, w,
            (w < 20 * li.AMU).astype(np.int32), tr, 1e4, beams=BEAMS, baths=BATHS, dt=li.DT,
            nsteps=20, ion_base=o)
        # the pair paths' force error over the run, with room for its growth, and roundings
        scale = np.max(oracle_mod.accel_scale(*part[:3], q, w, tr, 0.0))
        dv = 20 * 20 * li.DT * TOL[prec] * scale + 1e-12 * np.max(np.abs(part[3:]))
        for k, c in enumerate(("x", "y", "z", "vx", "vy", "vz")):
            tol = dv if k > 2 else 20 * li.DT * dv + 1e-13 * np.max(np.abs(part[:3]))
            assert np.max(np.abs(got[0][k][o:o + m] - ref[c])) <= tol, (m, c)
        o += m
