"""Cached tile choices are applied only while their numbers mean the kernels they
were timed on (no GPU)."""
from paper_1211_4461_amd import autotune


def test_key_holds_the_version_of_the_variants(monkeypatch):
    base = dict(arch="gfx950", tunable=3, dim=2, shape=(1023, 1023), n_dirs=0, precision=1, n_variants=3)
    now = autotune.key(**base)
    monkeypatch.setattr(autotune, "VARIANTS_VERSION", autotune.VARIANTS_VERSION + 1, raising=False)
    assert autotune.key(**base) != now


def test_choices_of_the_first_variants_are_not_applied():
    """The key of a choice made before the pre-smoothing tile heights, the 3D
    tiles and the tail variants came to mean other kernels."""
    opts = ",".join(f"{k}=0" for k in autotune.KEY_OPTIONS)
    old = f"gfx950|tunable=3|nv=3|d=2|m=1023x1023|M=0|prec=1|{opts}"
    assert autotune.key("gfx950", 3, 2, (1023, 1023), 0, 1, 3) != old
