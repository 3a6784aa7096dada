"""The test functions of the ionisation amplitudes along short and long axes.

Row by row against the oracle's recurrence: an axis shorter than the stretch of
potential that the kernel holds at a time and one of several stretches (256 and
512 cells), one wavenumber and more than one block of them.  Rounding errors of
the recurrence grow with its length, so the bar of the smoother grids (1e-11 at
256 cells) scales with it.
"""
import numpy as np
import pytest

from paper_1211_4461_amd import workloads as W
from tests.compare import elementwise

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("M", [0, 32])
@pytest.mark.parametrize("n", [256, 512])
def test_axis_lengths(n, M):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from oracle import ion
    from paper_1211_4461_amd import ffmg as ff
    w = W.ionization_2d(1.97849931, n=n)
    m = n - 1
    q = torch.zeros((m, m), dtype=torch.complex128, device="cuda")
    h = ff.mg_setup(2, [n] * 2, [0.0] * 2, [w.hi] * 2, w.gamma, q, k0=1.0)
    kn, k1, k2, _ = ion.wavenumbers(w.energy, -1.02145, max(M, 1))
    ks = [kn] + (list(k1) + list(k2) if M else [])
    assert len(ks) == 1 + 2 * M
    v1 = torch.from_numpy(np.ascontiguousarray(w.params["v1"], dtype=np.complex128)).cuda()
    T = ff.ion_test_functions(h, 0, v1, ks).cpu().numpy()
    To = ion.test_functions(n, 0.0, w.hi, w.gamma, w.params["v1"], ks)
    assert max(elementwise(T[i], To[i]) for i in range(len(ks))) <= 1e-11 * n / 256
    h.destroy()
