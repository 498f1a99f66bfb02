"""The two-level preconditioner with every number of column groups: an apply
to 17, 33, 48 or 64 columns against the same columns in blocks of 16, with one
block of 256 patches and with more. Tolerance 1e-5 max|z|: E Z is kept in
FP32 (2^-24 relative), and a last-bit change of w in front of it moves the
sums over all atoms by as much.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_06704_amd import workloads as wl  # noqa: E402


@pytest.mark.parametrize("edge", [9.0, 2.5])
@pytest.mark.parametrize("nf", [17, 33, 48, 64])
def test_groups(edge, nf):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    geo = wl.electrode_geometry("coarse", 8, 8, True, [10.0], [50.0], 60.0)
    print(f"[case] N={geo.n} edge {edge} columns {nf}", flush=True)
    S = cpm.System(geo.pos, geo.box, store=("f32",))
    S.precond_dc(0.083, 8.0)
    S.precond_coarse(edge)
    r = torch.tensor(np.random.default_rng(nf).standard_normal((nf, geo.n)), device="cuda")
    z = S.precond_apply(r)
    for c in range(0, nf, 16):
        zc = S.precond_apply(r[c:c + 16].contiguous())
        assert float((z[c:c + 16] - zc).abs().max()) <= 1e-5 * float(z.abs().max()), c
