"""Inputs at the ends of the range of a double in the allocation-free FP64 evaluation: the
one launch from the caller's arrays gives infinities and NaNs where the packed path (taken
when an output overlaps an input) gives them, and the same values elsewhere."""
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


def _run(torch, n, rows, overlap):
    from paper_1907_10514_amd import lion as L

    d = [torch.tensor(r, device="cuda") for r in rows]
    out = d[:3] if overlap else [torch.empty_like(d[0]) for _ in range(3)]
    L.lion_accel_noalloc(n, *[t.data_ptr() for t in d], 9.0, li.OMEGA, 0.24, li.R0, li.Z0,
                         li.KAPPA, 1e-8, L.LION_FP64, *[t.data_ptr() for t in out],
                         torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return np.array([t.cpu().numpy() for t in out])


@pytest.mark.parametrize("row,value", [
    (3, np.inf), (3, -np.inf), (3, np.nan), (3, 1e300), (3, 1e288), (3, -1e270), (3, 5e-324),
    (3, 1e-310), (3, -0.0), (4, np.inf), (4, np.nan), (4, 5e-324), (4, 1e308), (0, np.inf),
    (1, np.nan), (2, 1e155), (2, -1e300), (0, 1e-320)])
@pytest.mark.parametrize("n", [2, 300, 1025])
def test_like_the_packed_path(torch_gpu, n, row, value):
    rng = np.random.default_rng(n)
    rows = [*rng.normal(0, 1e-5 * n ** (1 / 3), (3, n)), rng.choice([1.0, 2.0], n) * li.E_CHARGE,
            np.full(n, li.REF_MASS)]
    for i in (n - 1, n // 3):  # the last ion pads the direct path's loads
        r = [a.copy() for a in rows]
        r[row][i] = value
        got, ref = _run(torch_gpu, n, r, False), _run(torch_gpu, n, r, True)
        fin = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[~fin & ~np.isnan(ref)], ref[~fin & ~np.isnan(ref)])
        # sums of n terms in another order, against the largest of the ion's components
        scale = np.max(np.abs(np.where(fin, ref, 0.0)), axis=0)
        cap = np.maximum(scale, np.median(scale))
        off = np.abs(np.where(fin, got, 0.0) - np.where(fin, ref, 0.0))
        assert np.all(off <= 4e-15 * n * cap + 1e-300)
