"""What mg_tune_get reports on an untuned handle is what runs on it: the split
far field's default is the last variant, which chooses the tiles per launch; it
can be read, set, timed and gone back to like the others.  The number of tail
variants is a property of the handle, not of the variant that is set."""
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


@pytest.mark.parametrize("prec", ["FF_BF16X3", "FF_BF16X6"])
def test_untuned_far_field_reports_its_rule(ff, prec):
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    q = 0.1 * torch.randn((127, 127), generator=g, device="cuda", dtype=torch.complex128)
    h = ff.mg_setup(2, [128, 128], [-3.0] * 2, [3.0] * 2, 0.5, q, k0=1.0,
                    options=ff.default_options(ff_precision=getattr(ff, prec)))
    nv = ff.mg_tune_variants(h)
    assert ff.mg_tune_get(h) == nv - 1
    eta, dirs = np.array([0.6, 0.8]), W.directions_2d(33)
    F = ff.farfield_map(h, eta, None, dirs)
    assert ff.mg_tune_get(h) == nv - 1
    for v in (0, nv - 1):
        ff.mg_tune_set(h, v)
        assert ff.mg_tune_get(h) == v
        assert np.array_equal(ff.farfield_map(h, eta, None, dirs), F)
    best, times = ff.mg_tune_farfield(h, eta, None, dirs, reps=2)
    assert len(times) == nv and all(t > 0 for t in times) and best == int(np.argmin(times))
    with pytest.raises(ff.FfmgError):
        ff.mg_tune_set(h, nv)
    h.destroy()


@pytest.mark.parametrize("n,coarsest", [((32, 32), 16), ((64, 64), 16), ((64, 16), 8), ((32, 32), 8)])
def test_tail_variants_do_not_depend_on_the_one_set(ff, n, coarsest):
    """A variant whose tail would hold fewer than two levels has none (a
    coarsest level of 225 points and 256 allowed); the others can still be set
    from it, and the tuner goes through all of them."""
    shape = (n[1] - 1, n[0] - 1)
    q = 0.1 * torch.ones(shape, device="cuda", dtype=torch.complex128)
    h = ff.mg_setup(2, list(n), [-0.05 * k for k in n], [0.05 * k for k in n], 0.5, q, k0=1.0,
                    options=ff.default_options(coarsest_n=coarsest))
    b, u = torch.ones_like(q), torch.zeros_like(q)
    assert ff.mg_tune_variants(h, ff.TUNE_TAIL) == 3
    for v in (2, 1, 0, 2, 0):
        ff.mg_tune_set(h, v, ff.TUNE_TAIL)
        assert ff.mg_tune_get(h, ff.TUNE_TAIL) == v
        assert ff.mg_tune_variants(h, ff.TUNE_TAIL) == 3
        ff.mg_profile_enable(h, 5)
        assert ff.mg_tune_variants(h, ff.TUNE_TAIL) == 3
        ff.mg_profile_enable(h, 0)
    best, times = ff.mg_tune_solve(h, b, u, tol=1e-8, reps=1, tunable=ff.TUNE_TAIL)
    assert len(times) == 3 and times[best] == min(times) and ff.mg_tune_get(h, ff.TUNE_TAIL) == best
    h.destroy()
