"""cpm_rhs's scratch for the structure factors' grids when device memory is
short. Other memory is taken first, so that the grids do not fit, or only a
few at a time: b must be the same to the bit with any number of grids at a
time (each frame's sums are its own), and b of the direct product (to 1e-12
max|b|, as the two paths agree everywhere) without any. The grids are back
when memory is and the scratch grows, and they leave room for what the same
system allocates after them.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MB = 1 << 20
BOX = np.array([101.0, 67.0, 90.5])
M, FRAMES = 12007, 40


def _cpm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    return cpm


def _inputs(n):
    rng = np.random.default_rng(11)
    dev = "cuda"
    return [torch.tensor(rng.random((FRAMES, M, 3)) * BOX, device=dev),
            torch.tensor(rng.choice([-1.0, 1.0], size=(FRAMES, M)), device=dev),
            torch.linspace(-0.5, 0.5, n, device=dev, dtype=torch.float64)]


def _leave(mb):
    """Take all device memory but mb; the tensors that hold it."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while True:
        take = torch.cuda.mem_get_info()[0] - mb * MB
        if take < 22 * MB:
            return held
        # in pieces: one allocation of all would need one range that large
        held.append(torch.empty(min(take, 32 << 30), dtype=torch.uint8, device="cuda"))


def _system(cpm, n=70):
    return cpm.System(np.random.default_rng(3).random((n, 3)) * BOX, BOX)


def test_few_grids_and_none():
    cpm = _cpm()
    S = _system(cpm)
    t = _inputs(S.n)
    want32, _ = S.rhs(t[0][:32], t[1][:32], t[2])
    want, qs = S.rhs(*t)
    S.close()
    direct = torch.empty_like(want)
    S = _system(cpm)
    for f in range(0, FRAMES, 4):   # the static scratch takes a few frames
        S.rhs_noalloc(t[0][f:f + 4].contiguous(), t[1][f:f + 4].contiguous(), t[2],
                      direct[f:f + 4], torch.empty(4, device="cuda", dtype=torch.float64))
    S.close()
    assert not torch.equal(want, direct)
    out = torch.empty_like(want), torch.empty_like(qs)
    part = [t[0][:32], t[1][:32], t[2], out[0][:32], out[1][:32]]
    for mb, grids in ((2000, True), (300, False)):
        print(f"[case] {mb} MB left", flush=True)
        S = _system(cpm)
        held = _leave(mb)
        S.rhs(*part)
        torch.cuda.synchronize()
        held.clear()
        torch.cuda.empty_cache()
        b = out[0][:32]
        if grids:
            assert torch.equal(b, want32)
        else:
            assert float((b - direct[:32]).abs().max()) <= 1e-12 * float(direct.abs().max())
            assert not torch.equal(b, want32)
        S.rhs(*t, *out)
        assert torch.equal(out[0], want)
        S.close()


def test_a_later_allocation_has_room():
    """The inverse of 2592 atoms (58 MB) after a right-hand side whose scratch
    with all 16 grids would leave 30 MB."""
    cpm = _cpm()
    from paper_2111_06704_amd import workloads as wl
    geo = wl.electrode_geometry("room", 18, 18, False, [35.0], [85.0], 120.0)
    rng = np.random.default_rng(5)
    t = [torch.tensor(rng.random((16, 12000, 3)) * np.asarray(geo.box), device="cuda"),
         torch.tensor(rng.choice([-1.0, 1.0], size=(16, 12000)), device="cuda"),
         torch.tensor(wl.electrode_potential(geo), device="cuda")]
    out = torch.empty((16, geo.n), device="cuda", dtype=torch.float64), \
        torch.empty(16, device="cuda", dtype=torch.float64)

    def system():
        S = cpm.System(geo.pos, geo.box)
        S.dprime()   # loads the solver
        S.matvec(torch.ones((64, S.n), device="cuda", dtype=torch.float64))   # its largest workspace
        return S

    S = system()
    before = S.describe()["device_bytes"]
    S.rhs(*t, *out)   # with ample memory
    scratch = (S.describe()["device_bytes"] - before) // MB
    want = out[0].clone()
    S.close()
    assert scratch > 250
    S = system()
    print(f"[case] scratch {scratch} MB, {scratch + 30} MB left", flush=True)
    held = _leave(scratch + 30)
    try:
        S.rhs(*t, *out)
        S.mi_build(tol=1e-13)
    finally:
        held.clear()
        torch.cuda.empty_cache()
    assert torch.equal(out[0], want)
    S.close()
