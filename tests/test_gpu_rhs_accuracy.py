"""How far b is from its sums in 80-bit arithmetic, with the structure factors
through the grid and as direct products (cpm_rhs_noalloc never takes the
grid): one frame of 12 000 ions and 38 000 k-vectors at twelve atoms. The grid
must be at least as close, and within 1e-14 max|b|: the window's aliasing is
2e-15 of |S|, the rounding of its sums the same order, the real-space part's
erfc table 1.2e-16 a pair.
"""
import ctypes
import math

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2111_06704_amd import workloads as wl  # noqa: E402

LD = np.longdouble
TWO_PI = 2 * np.arccos(LD(-1))
libm = ctypes.CDLL("libm.so.6")
libm.erfcl.restype, libm.erfcl.argtypes = ctypes.c_longdouble, [ctypes.c_longdouble]
erfc = np.frompyfunc(lambda x: libm.erfcl(ctypes.c_longdouble(x)), 1, 1)


def _cis(u, n):
    t = u[:, None] * np.asarray(n, dtype=LD)[None, :]
    t = (t - np.rint(t)) * TWO_PI
    return np.cos(t), np.sin(t)


def _exact(atoms, ipos, iq, box):
    """-sum over the ions (chi = 0) at the atoms, neutral frame, in long double."""
    beta, rcut, a = LD(wl.EWALD_SPLIT), wl.RCUT, LD(wl.GAUSS_INV_WIDTH)
    kmax = 2.0 * wl.EWALD_SPLIT * math.sqrt(math.log(1.0 / wl.KSPACE_EPS))
    L = np.asarray(box, dtype=LD)
    r, x, q = atoms.astype(LD), ipos.astype(LD), iq.astype(LD)
    nm = [int(math.floor(kmax * b / (2.0 * math.pi))) for b in box]
    nx, ny, nz = np.arange(nm[0] + 1), np.arange(-nm[1], nm[1] + 1), np.arange(-nm[2], nm[2] + 1)
    cx, sx = _cis(x[:, 0] / L[0], nx)
    cy, sy = _cis(x[:, 1] / L[1], ny)
    cz, sz = _cis(x[:, 2] / L[2], nz)
    ax, bx = _cis(r[:, 0] / L[0], nx)
    ay, by = _cis(r[:, 1] / L[1], ny)
    az, bz = _cis(r[:, 2] / L[2], nz)
    cz, sz = cz * q[:, None], sz * q[:, None]
    vol = L.prod()
    rec = np.zeros(len(r), dtype=LD)
    for i, n in enumerate(nx):
        K2 = (TWO_PI * LD(n) / L[0]) ** 2 + (TWO_PI * ny.astype(LD) / L[1])[:, None] ** 2 \
            + (TWO_PI * nz.astype(LD) / L[2])[None, :] ** 2
        k2 = (2.0 * math.pi) ** 2 * ((n / box[0]) ** 2 + (ny / box[1])[:, None] ** 2
                                     + (nz / box[2])[None, :] ** 2)
        half = (n > 0) | (ny[:, None] > 0) | ((ny[:, None] == 0) & (nz[None, :] > 0))
        on = half & (k2 <= kmax * kmax)
        keep = on.any(1)
        w = np.zeros(K2.shape, dtype=LD)
        w[on] = 2 * (2 * TWO_PI / vol) * np.exp(-K2[on] / (4 * beta * beta)) / K2[on]
        c = cx[:, i, None] * cy[:, keep] - sx[:, i, None] * sy[:, keep]
        s = sx[:, i, None] * cy[:, keep] + cx[:, i, None] * sy[:, keep]
        re = w[keep] * (c.T @ cz - s.T @ sz)
        im = w[keep] * (s.T @ cz + c.T @ sz)
        pc = ax[:, i, None] * ay[:, keep] - bx[:, i, None] * by[:, keep]
        ps = bx[:, i, None] * ay[:, keep] + ax[:, i, None] * by[:, keep]
        # sum over the column: Re(conj(P Z) G) = cos Re G + sin Im G
        for j in range(len(r)):
            cc = pc[j, :, None] * az[j] - ps[j, :, None] * bz[j]
            ss = ps[j, :, None] * az[j] + pc[j, :, None] * bz[j]
            rec[j] += (cc * re + ss * im).sum()
    real = np.zeros(len(r), dtype=LD)
    for j in range(len(r)):
        d = x - r[j]
        d -= L * np.rint(d / L)   # box edges above 2 rcut: one image at most
        d = np.sqrt((d * d).sum(1))
        near = d < rcut
        t = d[near]
        real[j] = (q[near] * (erfc(beta * t) - erfc(a * t)).astype(LD) / t).sum()
    return -(rec + real)


def test_grid_is_as_close_as_direct():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    geo = wl.electrode_geometry("accuracy", 18, 18, False, [35.0], [85.0], 120.0)
    assert min(geo.box) > 2 * wl.RCUT
    frames, m, f = 16, 12000, 3
    rng = np.random.default_rng(8)
    ipos = rng.random((frames, m, 3)) * geo.box
    ipos[:, :, 2] = 37.0 + 46.0 * rng.random((frames, m))
    iq = np.tile([1.0, -1.0], (frames, m // 2))
    S = cpm.System(geo.pos, geo.box, wl.GAUSS_INV_WIDTH, wl.EWALD_SPLIT, wl.RCUT, wl.KSPACE_EPS)
    dev = "cuda"
    t = [torch.tensor(v, device=dev) for v in (ipos, iq, np.zeros(geo.n))]
    b, _ = S.rhs(*t)
    bd, qd = torch.empty((1, geo.n), device=dev, dtype=torch.float64), \
        torch.empty(1, device=dev, dtype=torch.float64)
    S.rhs_noalloc(t[0][f:f + 1].contiguous(), t[1][f:f + 1].contiguous(), t[2], bd, qd)
    print(f"[case] N={geo.n}, {S.describe()['n_kvec']} k-vectors", flush=True)
    at = np.random.default_rng(9).permutation(geo.n)[:12]
    want = _exact(np.mod(geo.pos[at], geo.box), ipos[f], iq[f], np.asarray(geo.box))
    scale = np.max(np.abs(want))
    eg = float(np.max(np.abs(b[f].cpu().numpy()[at] - want)) / scale)
    ed = float(np.max(np.abs(bd[0].cpu().numpy()[at] - want)) / scale)
    print(f"[case] error of b: grid {eg:.1e}, direct {ed:.1e} of max|b|", flush=True)
    assert not torch.equal(b[f], bd[0])
    assert eg <= ed and eg <= 1e-14
