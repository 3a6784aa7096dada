"""The learned smoother's inference kernel where its tiles end.

One smoothing step against the oracle's network with BF16 activations, to the bar
of the smoother's own inference test (1e-2 of the update: BF16 rounding of
activations that differ in the last place): a grid of less than one tile, one
with no interior tile, and one where a workgroup goes through several tiles.
"""
import numpy as np
import pytest

from oracle import convnet as cn
from paper_1211_4461_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [16, 32, 512])
def test_learned_step_at_tile_edges(orc, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg as ff
    w = W.bumps_2d(n=n, seed=3, k0=1.5, M=8)
    Ws = [np.asarray(a * 0.7, dtype=np.complex64) for a in cn.init_weights(6)]
    h, _ = ff.setup_workload(w, options=ff.default_options(smoother=ff.SMOOTH_LEARNED, smoother_weights=Ws))
    g = orc.Grid(2, w.n, w.lo, w.hi)
    kappa, q, k0 = orc.problem(w.kind, w.k0, w.energy, w.coef)
    b = orc.rhs_plane_wave(g, w.gamma, k0, q, w.eta)
    r = np.random.default_rng(n)
    u0 = 0.1 * (r.standard_normal(g.shape) + 1j * r.standard_normal(g.shape))
    ud = torch.from_numpy(u0).cuda()
    ff.mg_learned_smooth(h, torch.from_numpy(np.ascontiguousarray(b, dtype=np.complex128)).cuda(), ud)
    torch.cuda.synchronize()
    upd = ud.cpu().numpy() - u0
    hh = (w.hi - w.lo) / w.n
    ref = cn.smooth_step(Ws, orc.residual(g, w.gamma, kappa, b, u0), kappa * hh * hh, hh * hh, quant=True)
    assert np.linalg.norm(upd - ref) / np.linalg.norm(ref) < 1e-2
