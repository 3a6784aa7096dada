"""The training kernel where its tiling can go wrong: one patch and counts that
do not fill the gradient sum's waves, the smallest and the largest border
(1 and 12), errors on either side of the growth penalty, data that is
nonzero only at the patch's corners; loss and gradients against the oracle with
the bars of the other training tests."""
import numpy as np
import pytest

from oracle import convnet as cn
from tests.compare import rel as relerr

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg
    ffmg.lib()
    return ffmg


def field(rng, count, scale, corners):
    a = (rng.standard_normal((count, 32, 32)) + 1j * rng.standard_normal((count, 32, 32))) * scale
    if corners:
        m = np.zeros((32, 32))
        m[[0, 0, 31, 31], [0, 31, 0, 31]] = 1.0
        a = a * m
    return a.astype(np.complex64)


@pytest.mark.parametrize("count,border,escale,corners",
                         [(1, 1, 0.3, False), (1, 12, 3.0, False), (3, 4, 0.01, False), (17, 8, 0.3, False),
                          (2, 1, 0.3, True)])
def test_loss_and_gradients(ff, count, border, escale, corners):
    rng = np.random.default_rng(count + 100 * border)
    rt, et = field(rng, count, 1.0, corners), field(rng, count, escale, corners)
    kt = field(rng, count, 0.05, False) + np.complex64(0.1)
    Ws = [w.astype(np.complex64).astype(np.complex128) for w in cn.init_weights(7)]
    net = ff.Net(Ws)
    L, G = net.loss_grad(*(torch.from_numpy(a).cuda() for a in (rt, kt, et)), border=border)
    mask = cn.interior_mask(32, 32, border)
    Lo, Go = 0.0, [np.zeros_like(w) for w in Ws]
    for p in range(count):
        Lp, gp = cn.loss_and_grads(Ws, *(a[p].astype(np.complex128) for a in (rt, kt, et)), mask, quant=True)
        Lo += Lp / count
        Go = [a + b / count for a, b in zip(Go, gp)]
    assert abs(L - Lo) <= 5e-3 * Lo, (L, Lo)
    for l in range(3):
        assert relerr(G[l], Go[l]) < 1e-2, (l, relerr(G[l], Go[l]))
