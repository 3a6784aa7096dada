"""Rules that choose kernel tiles on the host (no GPU)."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1211_4461_amd", "csrc")


@pytest.fixture(scope="module")
def rows(tmp_path_factory):
    """rows[fp32, N, variant] of the one-pass pre-smoothing tile."""
    d = tmp_path_factory.mktemp("tiles")
    cases = [(f, n, v) for f in (0, 1) for n in (961, 255 ** 2, 1023 ** 2, (1 << 21) - 1, 1 << 21, 2047 ** 2, 8191 ** 2)
             for v in (0, 1, 2)]
    body = "".join(f'printf("%d\\n", ffmg::presmooth_rows({f}, {n}u, {v}));\n' for f, n, v in cases)
    (d / "t.cpp").write_text(f'#include <cstdio>\n#include "ffmg_tiles.hpp"\nint main() {{\n{body}}}\n')
    subprocess.run(["g++", "-std=c++17", "-I" + CSRC, "-o", str(d / "t"), str(d / "t.cpp")], check=True)
    out = subprocess.run([str(d / "t")], check=True, capture_output=True, text=True).stdout.split()
    return dict(zip(cases, map(int, out)))


def test_presmoothing_variants_are_the_two_heights(rows):
    """Variants 0 and 2 differ on every finest level, so both heights can be
    selected and the tuner times no kernel twice."""
    for (f, n, v), r in rows.items():
        assert r in (8, 16)
        if v == 2:
            assert {rows[f, n, 0], r} == {8, 16}, (f, n)


def test_presmoothing_default_height(rows):
    for (f, n, v), r in rows.items():
        if v == 0:
            assert r == (16 if f and n >= 1 << 21 else 8), (f, n)
