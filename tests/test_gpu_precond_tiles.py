"""The block-dense apply z = P r at the edges of its tiling: fewer atoms than
one tile of 32, one atom past a full tile, ragged counts, every number of
column groups (16, 32, 48, 64 columns), and a system of more than 512 tiles
(its workgroups have half the waves).

Against the oracle's P: |z - z_o| <= 1e-12 max|z_o| as for the larger sizes.
The system of many tiles is a 6 x 6 repetition of a smaller periodic one whose
box exceeds 2 r_cut: its local matrices are those of the small system, so a
right-hand side repeated the same way gives the small system's z, to 1e-12
max|z| (the same sums in another order).
"""
import numpy as np
import pytest
from scipy.spatial import cKDTree

from oracle import precond as pc
from paper_2111_06704_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

A, G, RDC = wl.GAUSS_INV_WIDTH, 0.083, 8.0


def _cpm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    return cpm


@pytest.fixture(scope="module")
def ragged():
    cache = {}

    def get(n):
        if n not in cache:
            geo = wl.electrode_geometry("ragged", 6, 6, True, [10.0], [50.0], 60.0)
            keep = np.sort(np.random.default_rng(n).permutation(geo.n)[:n])
            print(f"[case] N={n}", flush=True)
            S = _cpm().System(geo.pos[keep], geo.box)
            S.precond_dc(G, RDC)
            cache[n] = S, pc.dc_preconditioner(geo.pos[keep], geo.box, A, G, RDC)
        return cache[n]

    return get


@pytest.mark.parametrize("n", [5, 32, 33, 275])
@pytest.mark.parametrize("nf", [1, 17, 48, 64])
def test_ragged_tiles(ragged, n, nf):
    S, P = ragged(n)
    r = np.random.default_rng(nf).standard_normal((nf, n))
    z = S.precond_apply(torch.tensor(r, device="cuda")).cpu().numpy()
    zo = r @ P.T
    assert np.max(np.abs(z - zo)) <= 1e-12 * np.max(np.abs(zo))


def test_many_tiles_repeat_the_small_system():
    cpm = _cpm()
    a, k, rc = 8, 6, 7.0
    small = wl.electrode_geometry("small", a, a, True, [10.0], [30.0], 45.0)
    large = wl.electrode_geometry("large", k * a, k * a, True, [10.0], [30.0], 45.0)
    assert min(small.box) > 2 * rc and (large.n + 31) // 32 > 512
    # atom of the small system that each atom of the large one repeats
    tree = cKDTree(np.mod(small.pos + 0.3, small.box), boxsize=small.box)
    d, src = tree.query(np.mod(large.pos + 0.3, small.box))
    assert d.max() < 1e-6
    Ss = cpm.System(small.pos, small.box)
    Ss.precond_dc(0.1, rc)
    print(f"[case] N={large.n}", flush=True)
    Sl = cpm.System(large.pos, large.box)
    Sl.precond_dc(0.1, rc)
    for nf in (16, 32, 48, 64):
        r = np.random.default_rng(nf).standard_normal((nf, small.n))
        zs = Ss.precond_apply(torch.tensor(r, device="cuda")).cpu().numpy()
        zl = Sl.precond_apply(torch.tensor(r[:, src].copy(), device="cuda")).cpu().numpy()
        assert np.max(np.abs(zl - zs[:, src])) <= 1e-12 * np.max(np.abs(zs))
