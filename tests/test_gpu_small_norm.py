"""The residual norm and the control update of a small level in one workgroup.

A plain solve against the reference kernel path, which takes the norm's pass and
the update as launches of their own: the same number of cycles, the same residual
and iterate, bit for bit, on levels of one tile of the norm's pass (64 x 16 points)
to four, square and long, and on the first with more.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("nx,ny", [(16, 16), (64, 16), (32, 64), (64, 64), (128, 32), (256, 16), (64, 128)])
def test_solve_equals_reference_path(nx, ny):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg as ff
    r = np.random.default_rng(nx + ny)
    q, b = (torch.from_numpy(r.standard_normal((ny - 1, nx - 1)) + 1j * r.standard_normal((ny - 1, nx - 1))).cuda()
            for _ in range(2))
    got = []
    for tile in (1, 0):
        h = ff.mg_setup(2, [nx, ny], [-5.0 * nx / 64, -5.0 * ny / 64], [5.0 * nx / 64, 5.0 * ny / 64], 0.5, 0.1 * q,
                        k0=1.0, options=ff.default_options(tile_config=tile, coarsest_n=4))
        u = torch.zeros_like(b)
        info = ff.mg_solve(h, b, u, tol=1e-11)
        torch.cuda.synchronize()
        assert info.status == 0 and info.cycles > 3
        got.append((info.cycles, info.rel_residual, u))
        h.destroy()
    assert got[0][:2] == got[1][:2]
    assert torch.equal(got[0][2], got[1][2])
