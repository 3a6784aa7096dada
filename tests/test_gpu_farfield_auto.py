"""Split-BF16 far fields whose contraction variant is chosen per launch equal
those of every explicit variant bit for bit: numbers of tiles on either side of
the rule's lines, one and several row tiles, ragged last tiles, 2D and 3D."""
import numpy as np
import pytest

from paper_1211_4461_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg
    ffmg.lib()
    return ffmg


@pytest.mark.parametrize("dim,n,M,polar", [(2, 64, 3, 0), (2, 1024, 500, 0), (2, 2048, 361, 0), (2, 2048, 790, 0),
                                           (3, 32, 5, 3), (3, 128, 9, 9), (3, 128, 40, 33), (3, 256, 2, 7),
                                           (3, 256, 3, 19), (3, 256, 130, 40)])
@pytest.mark.parametrize("parts", [2, 3])
def test_auto_variant_is_bitwise_every_variant(ff, dim, n, M, polar, parts):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + M)
    shape = (n - 1,) * dim
    q = 0.1 * torch.randn(shape, generator=g, device="cuda", dtype=torch.complex128)
    u = torch.randn(shape, generator=g, device="cuda", dtype=torch.complex128)
    dirs = W.directions_2d(M) if dim == 2 else W.directions_3d(M, polar)
    eta = np.array([0.6, 0.8, 0.0][:dim])
    h = ff.mg_setup(dim, [n] * dim, [-3.0] * dim, [3.0] * dim, 0.5, q, k0=1.0,
                    options=ff.default_options(ff_precision=ff.FF_BF16X6 if parts == 3 else ff.FF_BF16X3))
    F0 = ff.farfield_map(h, eta, u, dirs)
    for v in range(ff.mg_tune_variants(h, ff.TUNE_FF_GEMM)):
        ff.mg_tune_set(h, v, ff.TUNE_FF_GEMM)
        assert np.array_equal(F0, ff.farfield_map(h, eta, u, dirs)), v
    h.destroy()
