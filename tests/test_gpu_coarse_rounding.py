"""The coarsest operator's inverse holds to rounding also where one slice of the
grid is close to singular by itself: its columns, read as exact solves for unit
vectors on a one-level hierarchy, have max |A X - I| within a few eps ||A|| max |X|
(elimination with pivots over the whole matrix stays below 4; the inverse by
slices is let through up to 8 by real and imaginary part, and the sums of seven
terms here round by less than 7 more)."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

BOUND = 8 * math.sqrt(2.0) * math.sqrt(2.0) + 7   # moduli of r and of what its bound is made of


@pytest.fixture(scope="module")
def ff():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1211_4461_amd import ffmg
    ffmg.lib()
    return ffmg


def residual_of_inverse(ff, orc, n, q, gamma=math.pi / 6, k0=1.1):
    """max |A X - I| in units of eps ||A|| max |X|."""
    h = ff.mg_setup(len(n), list(n), [-4.0] * len(n), [4.0] * len(n), gamma, torch.from_numpy(q).cuda(), k0=k0,
                    options=ff.default_options(coarsest_n=min(n)))
    assert h.num_levels() == 1
    g = orc.Grid(len(n), n, -4.0, 4.0)
    kappa, _, _ = orc.problem(0, k0, 0.0, q)
    b = torch.zeros(q.shape, dtype=torch.complex128, device="cuda")
    u = torch.empty_like(b)
    r, x = 0.0, 0.0
    for j in range(q.size):
        b.zero_()
        b.view(-1)[j] = 1.0
        col = ff.mg_fmg(h, b, u, 1).cpu().numpy()
        r = max(r, np.abs(orc.residual(g, gamma, kappa, b.cpu().numpy(), col)).max())
        x = max(x, np.abs(col).max())
    h.destroy()
    norm = 4.0 * np.sum(1.0 / g.h ** 2) + np.abs(kappa).max()
    return r / (np.finfo(float).eps * norm * x)


@pytest.mark.parametrize("where", ["first", "middle"])
@pytest.mark.parametrize("n", [(4, 8), (8, 4), (8, 16), (16, 16), (4, 4, 8)])
def test_nearly_singular_slice(ff, orc, n, where):
    """The contrast of a slice (across the longest axis, the first of equal
    ones) cancels its diagonal up to a relative shift: an odd number of points
    in a line with zero diagonal is singular, the whole operator is not."""
    gamma, o = math.pi / 6, int(np.argmax(n))
    d = 2 * np.exp(-2j * gamma) * sum((k / 8.0) ** 2 for k in n) - 1.1 ** 2
    for shift in (1e-2, 1e-3, 1e-4, 1e-5, 1e-6, 1e-7, 1e-8):
        rng = np.random.default_rng(1)
        q = 0.3 * rng.standard_normal(tuple(k - 1 for k in n[::-1])) + 0j
        at = [slice(None)] * len(n)
        at[len(n) - 1 - o] = 0 if where == "first" else (n[o] - 1) // 2
        q[tuple(at)] = d * (1 + shift)
        assert residual_of_inverse(ff, orc, n, q, gamma) < BOUND, shift
