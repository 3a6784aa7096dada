"""The tiles of the two-sweep 3D pass, chosen by type and number of points.

A V-cycle of the default tiles against the single sweeps of the reference kernel
path, bit for bit: hierarchies whose finest level is on either side of the two
limits (2^17 and 2^20 points: 31^3 and 63^3, 63^3 and 127^3), with an even and an
odd number of sweeps (the pair and the single pass) and from a guess and from
zero, in both precisions and every variant.
"""
import numpy as np
import pytest

from paper_1211_4461_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nu", [2, 3])
@pytest.mark.parametrize("n", [16, 32, 64, 128])
def test_tiles_give_the_bits_of_single_sweeps(n, nu):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg as ff
    w = W.radial_3d(n, L=6.0, n_az=4, n_pol=3)
    r = np.random.default_rng(n)
    b, v0 = (torch.from_numpy(r.standard_normal((n - 1,) * 3) + 1j * r.standard_normal((n - 1,) * 3)).cuda()
             for _ in range(2))

    def cycles(prec, variant, tile):
        h, _ = ff.setup_workload(w, options=ff.default_options(nu1=nu, nu2=nu, precision=prec, tile_config=tile,
                                                               max_cycles=4))
        if variant is not None:
            ff.mg_tune_set(h, variant, ff.TUNE_SWEEP3D)
        v = v0.clone()
        ff.mg_vcycle(h, b, v)
        z = torch.zeros_like(b)
        info = ff.mg_solve(h, b, z, tol=1e-6, raise_on_noconv=False)
        torch.cuda.synchronize()
        h.destroy()
        return v, z, info.cycles

    for prec in (0, 1):
        ref = cycles(prec, None, 1)
        for variant in (None, 0, 1, 2, 3, 4):
            got = cycles(prec, variant, 0)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1]) and got[2] == ref[2], (prec, variant)
