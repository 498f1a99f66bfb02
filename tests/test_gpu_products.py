"""Block product V = E P at the edges of its tiles: row tiles of 128 (one, an
odd number, one more than full), k slices that hold unequal numbers of chunks,
and 32 / 48 / 64 columns (the wide kernels), against the stored E in FP64.

Tolerances, element by element relative to |E| |P|: FP64 1e-13 (at most 1152
additions of 2^-53 each); FP32 and BF16 storage 1e-5 (the matrix cores add at
most 128 entries in FP32, 128 x 2^-24 = 7.6e-6, before the sum moves to FP64;
the three-part operands are exact to 2^-24).
"""
import numpy as np
import pytest

from paper_2111_06704_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def systems():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    cache = {}

    def get(arm, zig):
        if (arm, zig) not in cache:
            geo = wl.electrode_geometry("edge", arm, zig, True, [10.0], [30.0], 45.0)
            print(f"[case] N={geo.n}", flush=True)
            cache[arm, zig] = cpm.System(geo.pos, geo.box, store=("f32", "bf16"))
        return cpm, cache[arm, zig]

    return get


@pytest.mark.parametrize("cells", [(2, 2), (4, 4), (3, 11), (6, 11), (8, 17)])
@pytest.mark.parametrize("nf", [17, 33, 49, 64, 81])
def test_wide_product(systems, cells, nf):
    cpm, S = systems(*cells)
    g = torch.Generator(device="cuda")
    g.manual_seed(nf + 1000 * cells[1])
    P = torch.randn((nf, S.n), generator=g, device="cuda", dtype=torch.float64)
    for prec, tol in ((cpm.PREC_F64, 1e-13), (cpm.PREC_F32, 1e-5), (cpm.PREC_BF16, 1e-5)):
        E = S.get_E(prec).double()
        Q = P if prec == cpm.PREC_F64 else P.float().double()
        V = S.matvec(P, prec)
        bound = tol * (Q.abs() @ E.abs().T.contiguous())
        assert torch.all((V - Q @ E.T.contiguous()).abs() <= bound)
