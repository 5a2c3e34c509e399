"""Allocation-free forces at the edges of their one-launch FP64 path (1, 2 and 4 targets
per workgroup, 5120 ions and above) and in the other precisions against the oracle; and
with outputs that overlap inputs, which the path of packed copies takes."""
from __future__ import annotations

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "mixed": 1e-6, "mixed_kahan": 1e-6}  # of the force scale


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


@pytest.mark.parametrize("prec", ["fp64", "mixed", "mixed_kahan"])
@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 1023, 1024, 1025, 2047, 5120, 5121])
@pytest.mark.parametrize("overlap", [False, True])
def test_accel_matches_oracle(torch_gpu, oracle_mod, n, prec, overlap):
    from paper_1907_10514_amd import lion as L

    torch = torch_gpu
    rng = np.random.default_rng(n)
    pos = rng.normal(0, 10e-6 * n ** (1 / 3), (3, n))
    if n > 2:
        pos[:, 1] = pos[:, 0]  # coincident: no force on each other
    charge = rng.choice([-1.0, 0.0, 1.0, 2.0], n) * li.E_CHARGE
    mass = rng.choice([17.0, 40.0], n) * li.AMU
    tr = oracle_mod.Trap(V0=9.0, Omega=li.OMEGA, U0=0.24, R0=li.R0, Z0=li.Z0, kappa=li.KAPPA)
    dev = [torch.tensor(a, dtype=torch.float64, device="cuda") for a in (*pos, charge, mass)]
    # one element past the boundary of 16 bytes: no wider alignment is asked for
    out = [torch.empty(n + 1, dtype=torch.float64, device="cuda")[1:] for _ in range(3)]
    if overlap:
        out[0], out[2] = dev[0], dev[4]
    L.lion_accel_noalloc(n, *[a.data_ptr() for a in dev], tr.V0, tr.Omega, tr.U0, tr.R0, tr.Z0,
                         tr.kappa, 3.7e-8, L.PRECISIONS[prec], *[a.data_ptr() for a in out],
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    got = np.array([a.cpu().numpy() for a in out])
    ref = np.array(oracle_mod.accel(*pos, charge, mass, tr, 3.7e-8))
    scale = oracle_mod.accel_scale(*pos, charge, mass, tr, 3.7e-8)
    assert np.all(np.sqrt(((got - ref) ** 2).sum(0)) <= TOL[prec] * scale)
