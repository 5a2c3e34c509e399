"""States through the pinned staging memory at the edges of its pieces (8192 ions): what
goes in comes out bit for bit, for one trap and for batches, and a NULL output is left
out."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest

import lion_inputs as li

pytestmark = pytest.mark.gpu
NAMES = ("x", "y", "z", "vx", "vy", "vz")


@pytest.fixture(scope="module")
def torch_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.cuda.set_device(0)
    return torch


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [1, 8191, 8192, 8193, 16384, 16385, 50001])
@pytest.mark.parametrize("batched", [False, True])
def test_state_round_trip(torch_gpu, n, prec, batched):
    from paper_1907_10514_amd import Simulation
    from paper_1907_10514_amd import lion as L

    rng = np.random.default_rng(n)
    sizes = [1000] * (n // 1000) + ([n % 1000] if n % 1000 else [])
    sim = Simulation(np.full(n, li.REF_MASS), np.zeros(n), prec, autotuned=False,
                     n_per_trap=sizes if batched else None)
    for _ in range(2):
        rows = rng.normal(0, 1e-4, (6, n))
        sim.set_state(*rows, 0.0)
        got, t = sim.get_state()
        assert t == 0.0
        for c, r in zip(NAMES, rows):
            assert np.array_equal(got[c], r), c
    y = np.full(n, 7.0)
    p = y.ctypes.data_as(ctypes.POINTER(ctypes.c_double))
    assert L.load().lion_get_state(sim.h, None, p, None, None, None, None, None) == L.LION_OK
    assert np.array_equal(y, rows[1])
    # neutral ions in no field coast: the second buffer of the stream is the state's own
    sim.step(3, 2.0 ** -26)
    got, _ = sim.get_state()
    x = rows[0].copy()
    for _ in range(3):
        x = x + 2.0 ** -26 * rows[3]
    assert np.array_equal(got["x"], x)
    sim.close()


def test_threads_share_the_staging_memory(torch_gpu):
    """Six threads, each with its own handle and stream, read and write states at once:
    more calls under way than idle blocks are kept."""
    import threading

    from paper_1907_10514_amd import Simulation

    torch, n, bad = torch_gpu, 20000, []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                sim = Simulation(np.full(n, li.REF_MASS), np.zeros(n), "fp64", autotuned=False)
                rng = np.random.default_rng(k)
                for _ in range(5):
                    rows = rng.normal(0, 1e-4, (6, n))
                    sim.set_state(*rows, 0.0)
                    got, _ = sim.get_state()
                    for c, r in zip(NAMES, rows):
                        if not np.array_equal(got[c], r):
                            bad.append((k, c))
                sim.close()
        except Exception as e:  # a thread's failure must reach the test
            bad.append((k, repr(e)))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
