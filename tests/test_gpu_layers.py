"""Back-projection through layers of electrode atoms against the oracle:
exact planes, layers of atoms that move (4 to 16 interpolation nodes each),
several slices of one thick layer, and atoms too scattered for layers, for
frame counts around the 16-frame tiles and atom counts around the 16-atom
tiles; ion counts around the 32-ion chunks of the structure factors, and one
group of ions against many. Tolerance as for b everywhere: 1e-12 max|b| (the
interpolation is chosen to 1e-17 of the sums).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ewald as ew  # noqa: E402

BETA, EPS, RCUT, A = 0.3, 1e-6, 9.0, 1.979
BOX = np.array([21.0, 24.0, 62.0])


def _b(pos, frames, m, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    rng = np.random.default_rng(seed)
    ipos = rng.random((frames, m, 3)) * BOX
    iq = rng.choice([-1.0, 1.0, 2.0], size=(frames, m))
    chi = rng.uniform(-0.5, 0.5, len(pos))
    S = cpm.System(pos, BOX, A, BETA, RCUT, EPS)
    t = [torch.tensor(x, device="cuda") for x in (ipos, iq, chi)]
    b, _ = S.rhs(*t)
    bo, _ = ew.rhs(pos, A, ipos, iq, chi, BOX, BETA, RCUT, ew.kmax_from_eps(BETA, EPS))
    err = np.max(np.abs(b.cpu().numpy() - bo))
    assert err <= 1e-12 * np.max(np.abs(bo)), err / np.max(np.abs(bo))
    b2, q2 = torch.empty_like(b), torch.empty(frames, device="cuda", dtype=torch.float64)
    S.rhs_noalloc(*t, b2, q2)
    err = np.max(np.abs(b2.cpu().numpy() - bo))
    assert err <= 1e-12 * np.max(np.abs(bo)), err / np.max(np.abs(bo))


def _layers(n, thick, seed):
    rng = np.random.default_rng(seed)
    z0 = np.array([1.0, 4.4, 57.0, 61.9])   # the last crosses the periodic boundary
    pos = rng.random((n, 3)) * BOX
    pos[:, 2] = (z0[np.arange(n) % 4] + (rng.random(n) - 0.5) * thick) % BOX[2]
    return pos


@pytest.mark.parametrize("thick", [0.0, 1e-9, 0.02, 0.3, 0.9, 2.5, 30.0])
@pytest.mark.parametrize("n,frames,m", [(200, 1, 33), (261, 16, 64), (1000, 17, 31), (203, 33, 1),
                                        (330, 5, 700)])
def test_layers(thick, n, frames, m):
    print(f"[case] thickness {thick} n {n} frames {frames} m {m}", flush=True)
    _b(_layers(n, thick, n), frames, m, n + m)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 64, 65, 129])
def test_few_atoms_and_many_planes(n):
    """n planes of one atom (exact up to 64), and none that pay beyond."""
    pos = np.random.default_rng(n).random((n, 3)) * BOX
    print(f"[case] {n} atoms at distinct z", flush=True)
    _b(pos, 3, 100, n + 1000)   # another seed: no ion on an atom
