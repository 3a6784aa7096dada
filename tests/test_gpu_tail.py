"""The one-workgroup tail on the shapes its layout distinguishes: one, two and
four rows a thread, rows of more and fewer than 64 points, 512 and 1024
threads, the finest level inside the tail.  Every iterate equals that of the
grid-wide kernels (tile_config 2) bit for bit."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg
    ffmg.lib()
    return ffmg


SHAPES = [((16, 16), 8), ((32, 32), 8), ((64, 64), 8), ((128, 128), 8), ((64, 32), 8), ((128, 64), 8), ((64, 128), 8),
          ((64, 16), 8), ((16, 64), 8), ((64, 64), 4), ((128, 8), 4), ((8, 128), 4), ((128, 16), 4), ((16, 128), 4),
          ((256, 32), 4), ((64, 64), 16), ((128, 64), 16)]


@pytest.mark.parametrize("n,coarsest", SHAPES)
def test_tail_is_bitwise_the_grid_wide_cycle(ff, n, coarsest):
    lo, hi = [-0.05 * k for k in n], [0.05 * k for k in n]
    shape = (n[1] - 1, n[0] - 1)
    rng = np.random.default_rng(n[0] + 3 * n[1])
    coef = torch.from_numpy(0.4 * (rng.random(shape) + 0.3j * rng.random(shape))).cuda()
    b = torch.from_numpy(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).cuda()

    def run(tile_config, prec, nu):
        h = ff.mg_setup(2, list(n), lo, hi, math.pi / 6, coef, k0=0.9,
                        options=ff.default_options(tile_config=tile_config, precision=prec, coarsest_n=coarsest, nu1=nu,
                                                   nu2=3 - nu if nu != 2 else 2, max_cycles=3))
        out = [ff.mg_fmg(h, b, torch.empty_like(b), k).clone() for k in (0, 2)]
        u = torch.zeros_like(b)
        for _ in range(2):
            out.append(ff.mg_vcycle(h, b, u).clone())
        u.zero_()
        info = ff.mg_solve(h, b, u, tol=1e-14, raise_on_noconv=False)
        torch.cuda.synchronize()
        h.destroy()
        return out + [u], info.rel_residual

    for prec in (ff.FP64, ff.FP32_IR):
        for nu in (1, 2, 3, 0):
            (got, r0), (ref, r1) = run(0, prec, nu), run(2, prec, nu)
            for k, (x, y) in enumerate(zip(got, ref)):
                assert torch.equal(x, y), (prec, nu, k)
            assert r0 == r1, (prec, nu)
