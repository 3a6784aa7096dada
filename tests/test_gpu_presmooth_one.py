"""One pre-smoothing sweep, residual and full weighting as one 2D pass.

V-cycle iterates (from a guess on the finest level, from zero below) and a solve
with nu1 = 1 against the two launches and against the reference kernel path, bit
for bit: a level of less than a tile, of whole tiles less one point and of several
tiles, both tile heights, both precisions, with one and two sweeps after.
"""
import numpy as np
import pytest

from paper_1211_4461_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nu2", [1, 2])
@pytest.mark.parametrize("n", [16, 64, 256])
def test_one_sweep_pass_equals_two_launches(n, nu2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg as ff
    w = W.bumps_2d(n=n, seed=4, k0=1.0, M=8)
    r = np.random.default_rng(n)
    b, v0 = (torch.from_numpy(r.standard_normal((n - 1,) * 2) + 1j * r.standard_normal((n - 1,) * 2)).cuda()
             for _ in range(2))

    def run(prec, pre, tile):
        h, _ = ff.setup_workload(w, options=ff.default_options(nu1=1, nu2=nu2, precision=prec, tile_config=tile,
                                                               coarsest_n=8, max_cycles=5))
        if pre is not None:
            ff.mg_tune_set(h, pre, ff.TUNE_PRE)
            ff.mg_tune_set(h, 1, ff.TUNE_TAIL) if ff.mg_tune_variants(h, ff.TUNE_TAIL) > 1 else None
        v = v0.clone()
        ff.mg_vcycle(h, b, v)
        z = torch.zeros_like(b)
        info = ff.mg_solve(h, b, z, tol=1e-12, raise_on_noconv=False)
        torch.cuda.synchronize()
        h.destroy()
        return v, z, info.cycles

    for prec in (0, 1):
        ref = run(prec, None, 1)
        for pre in (None, 0, 1, 2):
            got = run(prec, pre, 0)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]) and got[2] == ref[2], (prec, pre)
