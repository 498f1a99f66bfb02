"""Coincident atoms are found through a grid of 2 A cells in which a pair is
only looked for across a face that both are near: pairs displaced by less and
by more than the 1e-6 A limit, along one and three axes, over cell faces, box
faces and corners, in boxes of one, two and many cells per edge. Host-side
validation: refused with CPM_EINVAL before any device call (accepted positions
go on to the device, which may not be there)."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("box", [(1.5, 3.0, 40.0), (4.0, 4.2, 5.9), (31.7, 22.0, 700.0)])
@pytest.mark.parametrize("axes", [(1, 0, 0), (0, 1, 0), (0, 0, 1), (1, 1, 1)])
@pytest.mark.parametrize("shift,bad", [(4e-7, True), (9.9e-7, True), (1.01e-6, False), (3e-6, False)])
def test_pairs_at_the_limit(box, axes, shift, bad):
    from paper_2111_06704_amd import cpm
    L = cpm.lib()
    p = cpm.Params(gauss_inv_width=1.979, ewald_split=0.3, rcut=2.0, kspace_eps=1e-6)
    b = np.array(box)
    nc = np.maximum(1, np.minimum(256, (b / 2.0).astype(int)))
    d = np.array(axes) / np.linalg.norm(axes) * shift
    starts = [b * 0.37, np.zeros(3), b - 2e-7, b / nc - 3e-7, b / nc * (nc // 2), b / nc * (nc - 1) - 5e-7,
              np.array([0.0, b[1] * 0.3, b[2] - 1e-9])]
    rng = np.random.default_rng(1)
    far = rng.random((20, 3)) * b
    for s in starts:
        for sign in (1.0, -1.0):
            pos = np.ascontiguousarray(np.vstack([far, s[None], (s + sign * d)[None]]))
            out = ctypes.c_void_p()
            rc = L.cpm_build_E(pos.ctypes.data, len(pos), b.ctypes.data, ctypes.byref(p), None,
                               ctypes.byref(out))
            if out.value:
                L.cpm_free(out)
            if bad:
                assert rc == cpm.CPM_EINVAL and b"coincide" in L.cpm_last_error(), (s, sign)
            else:
                assert rc != cpm.CPM_EINVAL, (s, sign)
