"""The reciprocal contraction's k range in parts (planes added to E by the
last pass), for tile counts from one to 45 and column counts from less than a
stage per part to many, against the oracle; E exactly symmetric and its FP32
copy its rounding. Tolerance as for E everywhere: 1e-12 max|E|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from oracle import ewald as ew  # noqa: E402

A, BETA, RC = 1.979, 0.3, 8.0


@pytest.mark.parametrize("n", [1, 127, 129, 300, 513, 1100])
@pytest.mark.parametrize("box,kmax", [((9.0, 8.3, 7.5), 1.0), ((24.0, 21.0, 40.0), 2.2)])
def test_E(n, box, kmax):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2111_06704_amd import cpm
    L = np.array(box)
    rng = np.random.default_rng(n)
    pos = rng.random((n, 3)) * L
    print(f"[case] n {n} box {box} kmax {kmax}", flush=True)
    S = cpm.System(pos, L, A, BETA, RC, 1e-6, kmax_override=kmax, store=("f32",))
    E = S.get_E().cpu().numpy()
    Eo = ew.ewald_matrix(pos, L, A, BETA, RC, kmax)
    assert np.max(np.abs(E - Eo)) <= 1e-12 * np.max(np.abs(Eo))
    assert np.array_equal(E, E.T)
    assert np.array_equal(S.get_E(cpm.PREC_F32).cpu().numpy(), E.astype(np.float32))
