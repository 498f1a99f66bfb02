"""Real-space part of the right-hand side where its image lists can go wrong,
against the oracle: boxes narrower than the cutoff (an ion is listed once per
image), tiles of atoms across a box face, lists that end at, before and after
64 images, one ion, ions on atoms, outside the box and on its faces, one ion
group and many, narrow and broad atoms (erfc(a d) over its whole range), and
the cell list (from 8192 ions). Tolerance as for b everywhere: 1e-12 max|b|.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ewald as ew  # noqa: E402

BETA, EPS = 0.3, 1e-6


@pytest.mark.parametrize("box", [(11.0, 7.5, 26.0), (40.0, 13.0, 9.0), (60.0, 52.0, 33.0)])
@pytest.mark.parametrize("n,m,frames", [(1, 1, 1), (64, 16, 2), (65, 17, 1), (130, 63, 3),
                                        (257, 64, 1), (63, 65, 5), (70, 129, 1), (200, 1000, 2),
                                        (129, 8195, 2)])
@pytest.mark.parametrize("rcut", [12.0, 6.5])
def test_image_lists(box, n, m, frames, rcut):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    rng = np.random.default_rng(n * 1000 + m)
    L = np.array(box)
    pos = rng.random((n, 3)) * L
    a = rng.uniform(0.35, 2.5, n)
    ipos = rng.random((frames, m, 3)) * L
    iq = rng.choice([-1.0, 1.0, 2.0], size=(frames, m))
    if m >= 16:
        ipos[:, 0] = pos[0]                       # on an atom, and close to an image of one
        ipos[:, 1] = pos[-1] + L * np.array([1, 0, -1]) + 0.1
        ipos[:, 2:6] = np.array([[0, 0, 0], [1, 1, 1], [0, 1, 0.5], [1, 0.25, 0]]) * L
        ipos[:, 6:9] += np.array([[1, -2, 3], [-1, 1, 0], [0, 0, 1]]) * L
    chi = rng.uniform(-0.5, 0.5, n)
    print(f"[case] box {box} n {n} m {m} frames {frames} rcut {rcut}", flush=True)
    S = cpm.System(pos, L, float(np.max(a)), BETA, rcut, EPS,
                   per_atom_width=a)
    t = lambda x: torch.tensor(x, device="cuda")   # noqa: E731
    b, qs = S.rhs(t(ipos), t(iq), t(chi))
    bo, qo = ew.rhs(pos, a, ipos, iq, chi, L, BETA, rcut, ew.kmax_from_eps(BETA, EPS))
    if m >= 16:   # the oracle leaves out d = 0; the limit of its summand there
        bo[:, 0] -= iq[:, 0] * 2.0 * (a[0] - BETA) / np.sqrt(np.pi)
    assert np.max(np.abs(b.cpu().numpy() - bo)) <= 1e-12 * np.max(np.abs(bo))
    assert np.array_equal(qs.cpu().numpy(), qo)
