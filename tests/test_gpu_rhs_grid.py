"""Structure factors through a grid (chosen for many ions and k-vectors)
against the direct path: cpm_rhs_noalloc never takes the grid, so the two
entry points evaluate the same sums in different ways. Tolerance as for b
everywhere: 1e-12 max|b| (the window's aliasing is 2e-15 of |S|, the direct
phases' rounding 5e-15).

Boxes: grids of the smallest edge (32 points, box edge shorter than the
cutoff's image range), edges that round up to a tile by much and by little,
more than 47 vectors along z (two passes of the z transform, and the
three-term recurrence on the direct side). Ions on box faces, outside the box
and on the corners of grid tiles; counts from the least that has a cell list.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _system(box, slab=False):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    rng = np.random.default_rng(3)
    n = 70
    pos = rng.random((n, 3)) * np.array(box)
    print(f"[case] box {box}", flush=True)
    return cpm.System(pos, np.array(box), slab=slab)


def _both(S, pos, q):
    dev = "cuda"
    p, c = torch.tensor(pos, device=dev), torch.tensor(q, device=dev)
    chi = torch.linspace(-0.5, 0.5, S.n, device=dev, dtype=torch.float64)
    b, qs = S.rhs(p, c, chi)
    b2, qs2 = torch.empty_like(b), torch.empty_like(qs)
    S.rhs_noalloc(p, c, chi, b2, qs2)
    assert torch.equal(qs, qs2)
    return b.cpu().numpy(), b2.cpu().numpy()


@pytest.mark.parametrize("box,m,frames", [((300.0, 14.0, 150.0), 8192, 12),
                                          ((90.0, 88.0, 61.0), 8201, 5),
                                          ((70.0, 110.0, 160.0), 9000, 2),
                                          ((101.0, 67.0, 90.5), 12007, 7)])
@pytest.mark.parametrize("slab", [False, True])
def test_grid_matches_direct(box, m, frames, slab):
    S = _system(box, slab)
    rng = np.random.default_rng(m)
    L = np.array(box)
    pos = rng.random((frames, m, 3)) * L
    q = rng.choice([-1.0, 1.0, 2.0], size=(frames, m))
    pos[:, :4] = np.array([[0, 0, 0], [1, 1, 1], [0, 1, 0.5], [1, 0.25, 0]]) * L   # faces
    pos[:, 4:8] += np.array([[1, -2, 3], [-1, 1, 0], [5, 5, -7], [0, 0, 1]]) * L    # images
    pos[:, 8:24] = (np.arange(16)[:, None] / 16.0) * L                             # tile corners
    b, bd = _both(S, pos, q)
    assert np.max(np.abs(b - bd)) <= 1e-12 * np.max(np.abs(bd))
    assert not np.array_equal(b, bd)   # the direct path would repeat itself to the bit


def test_dense_spot_and_empty_space():
    """All ions of a frame in one grid tile (long lists, mostly empty tiles)."""
    S = _system((90.0, 88.0, 61.0))
    rng = np.random.default_rng(5)
    pos = rng.random((9, 8300, 3)) * 5.0 + np.array([80.0, 2.0, 55.0])
    q = rng.choice([-1.0, 1.0], size=(9, 8300))
    b, bd = _both(S, pos, q)
    assert np.max(np.abs(b - bd)) <= 1e-12 * np.max(np.abs(bd))
    assert not np.array_equal(b, bd)


def test_not_a_number_stays_in_its_frame():
    S = _system((90.0, 88.0, 61.0))
    rng = np.random.default_rng(6)
    pos = rng.random((9, 8200, 3)) * np.array([90.0, 88.0, 61.0])
    q = rng.choice([-1.0, 1.0], size=(9, 8200))
    ref, _ = _both(S, pos, q)
    pos[1, 77, 2] = np.nan
    dev = "cuda"
    chi = torch.linspace(-0.5, 0.5, S.n, device=dev, dtype=torch.float64)
    b, _ = S.rhs(torch.tensor(pos, device=dev), torch.tensor(q, device=dev), chi)
    b = b.cpu().numpy()
    assert np.isnan(b[1]).all()
    assert np.array_equal(b[0], ref[0]) and np.array_equal(b[2:], ref[2:])
