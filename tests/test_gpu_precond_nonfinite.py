"""z = P r with a NaN or an infinity in r: it reaches the rows whose pattern
holds its atom and no others, although the product runs over tiles of rows
with zeros between the pattern's entries. The other rows are as without it,
to 1e-12 max|z| of the finite entries (the sums may run in another order).
"""
import numpy as np
import pytest

from oracle import precond as pc
from paper_2111_06704_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [33, 275])
@pytest.mark.parametrize("nf", [1, 17, 48])
def test_stays_in_its_pattern(n, nf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    geo = wl.electrode_geometry("ragged", 6, 6, True, [10.0], [50.0], 60.0)
    keep = np.sort(np.random.default_rng(n).permutation(geo.n)[:n])
    print(f"[case] N={n} columns {nf}", flush=True)
    S = cpm.System(geo.pos[keep], geo.box)
    S.precond_dc(0.083, 5.0)
    pattern = pc.dc_preconditioner(geo.pos[keep], geo.box, wl.GAUSS_INV_WIDTH, 0.083, 5.0) != 0.0
    rng = np.random.default_rng(nf)
    r = rng.standard_normal((nf, n))
    want = S.precond_apply(torch.tensor(r, device="cuda")).cpu().numpy()
    bad = {0: [(3, np.nan)], nf // 2: [(n - 1, np.inf), (0, -np.inf)], nf - 1: [(n // 2, np.inf)]}
    reached = np.zeros((nf, n), dtype=bool)
    for c, entries in bad.items():
        r0 = r[c].copy()
        for i, v in entries:
            r[c, i] = v
            r0[i] = 0.0
            reached[c] |= pattern[:, i]
        want[c] = S.precond_apply(torch.tensor(r0[None], device="cuda")).cpu().numpy()[0]
    z = S.precond_apply(torch.tensor(r, device="cuda")).cpu().numpy()
    assert not reached.all(axis=1).any()
    assert not np.isfinite(z[reached]).any()
    assert np.max(np.abs(z - want)[~reached]) <= 1e-12 * np.max(np.abs(want))
