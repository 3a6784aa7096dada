"""The FP64 far field on every branch of its contraction: blocks of two, four
and eight row tiles that form the integrand themselves, several row blocks over
a stored integrand, the split over k-steps; ragged numbers of directions, with
and without a scattered wave.  Reference: the same sum as dense products in
float64 (torch)."""
import math

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


def reference(n, L, gamma, k0, q, eta, u, dirs):
    dim = len(n)
    ax = [np.exp(1j * gamma) * (-L + 2 * L / m * torch.arange(1, m, dtype=torch.float64, device="cuda")) for m in n]
    ax = [a.to(torch.complex128) for a in ax]
    shape = lambda v, k: v.reshape([-1 if dim - 1 - d == k else 1 for d in range(dim)])
    uin = 1.0
    for k in range(dim):
        uin = uin * shape(torch.exp(1j * k0 * eta[k] * ax[k]), k)
    s = q * (uin if u is None else uin + u)
    E = [torch.exp(-1j * k0 * torch.from_numpy(np.ascontiguousarray(dirs[:, k])).cuda()[:, None] * ax[k][None])
         for k in range(dim)]
    out = []
    if dim == 2:
        out.append(((E[0] @ s.T) * E[1]).sum(-1))
    else:
        z, inv = np.unique(dirs[:, 2], return_inverse=True)
        for g in range(len(z)):
            i = np.where(inv == g)[0]
            t = (E[2][i[0]] @ s.reshape(s.shape[0], -1)).reshape(s.shape[1:])
            out.append(((E[0][i] @ t.T) * E[1][i]).sum(-1))
        order = np.argsort(np.concatenate([np.where(inv == g)[0] for g in range(len(z))]), kind="stable")
    F = torch.cat(out)
    if dim == 3:
        F = F[torch.from_numpy(order).cuda()]
    return F * np.exp(1j * dim * gamma) * np.prod([2 * L / m for m in n])


CASES = [(2, 64, 1, 0), (2, 64, 33, 0), (2, 256, 17, 0), (2, 2048, 250, 0), (2, 2048, 801, 0),
         (3, 32, 5, 9), (3, 256, 3, 4), (3, 256, 2, 17), (3, 256, 1, 33), (3, 256, 3, 40), (3, 256, 1, 70)]


@pytest.mark.parametrize("dim,n,M,polar", CASES)
def test_fp64_map(ff, dim, n, M, polar):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + M)
    shape = (n - 1,) * dim
    rnd = lambda: torch.randn(shape, generator=g, device="cuda", dtype=torch.complex128)
    q, u = 0.1 * rnd(), rnd()
    L, gamma, k0 = 3.0, 0.5, 1.1
    eta = np.array([0.6, 0.8, 0.0][:dim])
    dirs = W.directions_2d(M) if dim == 2 else W.directions_3d(M, polar)
    h = ff.mg_setup(dim, [n] * dim, [-L] * dim, [L] * dim, gamma, q, k0=k0, options=ff.default_options())
    for v in (u, None):
        F = torch.from_numpy(ff.farfield_map(h, eta, v, dirs)).cuda()
        ref = reference([n] * dim, L, gamma, k0, q, eta, v, dirs)
        # random signs: the terms add up to about sqrt(N) of their size, so the
        # relative error of two orders of summation is a few hundred eps at most
        assert (torch.linalg.vector_norm(F - ref) / torch.linalg.vector_norm(ref)).item() < 1e-12
    h.destroy()
