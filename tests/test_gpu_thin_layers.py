"""Layers of electrode atoms a few last bits of z thick (one plane computed in
two ways) beside a layer whose atoms move, against the oracle: the
interpolation nodes of such a layer have to stay apart although its atoms
hold only two to a few values of z. Tolerance as for b everywhere: 1e-12
max|b| (the interpolation is chosen to 1e-17 of the sums).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ewald as ew  # noqa: E402

BETA, EPS, RCUT, A = 0.3, 1e-6, 9.0, 1.979
BOX = np.array([21.0, 24.0, 62.0])


# thickness in units of the last bit of z (2^33 of them: 3e-5 A at 50 A)
@pytest.mark.parametrize("bits", [1, 2, 3, 5, 1 << 10, 1 << 20, 1 << 33])
@pytest.mark.parametrize("frames", [1, 17])
def test_last_bits(bits, frames):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    print(f"[case] {bits} last bits, {frames} frames", flush=True)
    rng = np.random.default_rng(bits % 1000 + frames)
    n = 500
    pos = rng.random((n, 3)) * BOX
    z0 = np.array([1e-3, 12.3, 25.0, 46.7, 55.1])[np.arange(n) % 5]
    pos[:, 2] = z0 + np.spacing(z0) * rng.integers(0, bits + 1, n)
    move = np.arange(n) % 5 == 4   # more than 64 distinct z
    pos[move, 2] += 0.02 * rng.random(move.sum())
    m = 100
    ipos = rng.random((frames, m, 3)) * BOX
    iq = rng.choice([-1.0, 1.0, 2.0], size=(frames, m))
    chi = rng.uniform(-0.5, 0.5, n)
    S = cpm.System(pos, BOX, A, BETA, RCUT, EPS)
    b, _ = S.rhs(*[torch.tensor(x, device="cuda") for x in (ipos, iq, chi)])
    bo, _ = ew.rhs(pos, A, ipos, iq, chi, BOX, BETA, RCUT, ew.kmax_from_eps(BETA, EPS))
    err = np.max(np.abs(b.cpu().numpy() - bo))
    assert err <= 1e-12 * np.max(np.abs(bo)), err / np.max(np.abs(bo))
