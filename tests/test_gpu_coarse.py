"""The coarsest operator's exact inverse on one-level hierarchies: slices along
each axis, slice sizes from 3 to 49 points, a chain of 63 slices, and operators
whose first slice alone is singular (the inverse by slices has to give way to
elimination with pivots over the whole matrix)."""
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


SHAPES = [(4, 4), (8, 8), (16, 8), (8, 16), (16, 16), (32, 32), (16, 64), (64, 16), (4, 256), (4, 4, 4), (8, 8, 8),
          (16, 8, 8), (8, 16, 8), (8, 8, 16), (16, 4, 16), (4, 4, 64), (64, 4, 4)]


def one_level(ff, n, q, gamma=math.pi / 6):
    return ff.mg_setup(len(n), list(n), [-4.0] * len(n), [4.0] * len(n), gamma, torch.from_numpy(q).cuda(), k0=1.1,
                       options=ff.default_options(coarsest_n=min(n)))


def solve_error(ff, orc, n, q, gamma=math.pi / 6):
    """||b - A u|| / (||A||_1 ||u||) for the exact solve's u."""
    h = one_level(ff, n, q, gamma)
    assert h.num_levels() == 1
    rng = np.random.default_rng(3)
    b = rng.standard_normal(q.shape) + 1j * rng.standard_normal(q.shape)
    u = ff.mg_fmg(h, torch.from_numpy(b).cuda(), torch.empty(q.shape, dtype=torch.complex128, device="cuda"), 1)
    u = u.cpu().numpy()
    h.destroy()
    g = orc.Grid(len(n), n, -4.0, 4.0)
    kappa, _, _ = orc.problem(0, 1.1, 0.0, q)
    norm = 4.0 * np.sum(1.0 / g.h ** 2) + np.abs(kappa).max()
    return np.linalg.norm(orc.residual(g, gamma, kappa, b, u)) / (norm * np.linalg.norm(u))


@pytest.mark.parametrize("n", SHAPES)
def test_exact_solve(ff, orc, n):
    rng = np.random.default_rng(sum(n))
    shape = tuple(k - 1 for k in n[::-1])
    q = 0.5 * (rng.standard_normal(shape) + 1j * rng.standard_normal(shape))
    # the backward error of an explicit inverse: n eps times a condition number, here at most a few hundred
    assert solve_error(ff, orc, n, q) < 1e-11


@pytest.mark.parametrize("n", [(4, 8), (8, 16), (32, 32)])
def test_singular_first_slice(ff, orc, n):
    """The contrast cancels the diagonal of the first slice: a chain of an odd
    number of points with zero diagonal is singular, the whole operator not."""
    gamma = math.pi / 6
    h = [8.0 / k for k in n]
    rng = np.random.default_rng(1)
    q = 0.3 * (rng.standard_normal((n[1] - 1, n[0] - 1)) + 0j)
    d = 2 * np.exp(-2j * gamma) * sum(1 / v ** 2 for v in h) - 1.1 ** 2
    q[0, :] = d
    assert solve_error(ff, orc, n, q, gamma) < 1e-11
