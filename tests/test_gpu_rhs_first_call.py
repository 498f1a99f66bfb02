"""The first right-hand side on a system whose structure factors go through
the grid: what it takes beyond a later call (the tables of the grid and the
scratch) is host work and allocation below 1.5 ms. With the window's
constants and the transform matrices made on the host for every system it
was 3 to 4 ms, more than such a call itself. The median over five systems,
after one that loads the code.
"""
import time

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def test_first_call_is_not_far_from_the_next():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    box = np.array([101.0, 67.0, 90.5])
    rng = np.random.default_rng(7)
    m, frames, n = 12007, 7, 70
    dev = "cuda"
    ipos = torch.tensor(rng.random((frames, m, 3)) * box, device=dev)
    iq = torch.tensor(rng.choice([-1.0, 1.0], size=(frames, m)), device=dev)
    chi = torch.zeros(n, device=dev, dtype=torch.float64)
    extra = []
    for _ in range(6):
        S = cpm.System(rng.random((n, 3)) * box, box)
        t = []
        for _ in range(2):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            S.rhs(ipos, iq, chi)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - t0)
        extra.append(t[0] - t[1])
        S.close()
    print(f"[case] first call beyond the second (ms): {[round(1e3 * x, 2) for x in extra]}", flush=True)
    assert np.median(extra[1:]) < 1.5e-3
