"""The choice of a draw behind a parallel prefix sum, on the CPU: the library's own functions (csrc/draw.hpp) behind a model of
the GPU's scan.  Its fp32 sums are not monotone, so the points drawn at are the ones where that shows: the sums themselves, and
the largest uniform numbers.  Whatever the sums do the element is one of the range, has mass, and covers the point as the
64-bit sums have it."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent
# An fp32 sum of this depth (stretch, six shuffle steps, sixteen waves: under 32 additions of positive terms) is within
# 32 x 2^-24 of the total; the point u * total of that total and the sum it is compared with both carry it.
EPS = 64 * 2.0 ** -24


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    out = tmp_path_factory.mktemp("draw") / "libdraw_model.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-o", str(out),
                    str(HERE / "draw_model.cpp")], check=True)
    fn = ctypes.CDLL(str(out)).draw_model
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_float, ctypes.c_void_p]
    fn.restype = ctypes.c_int

    def draw(mass, unit, u):
        rest = ctypes.c_float(0.0)
        at = fn(mass.ctypes.data, len(mass), unit, float(u), ctypes.byref(rest))
        return at, rest.value
    return draw


def masses(rng, n, kind):
    if kind == "flat":
        m = rng.random(n) + 0.5
    else:
        m = np.exp(-40.0 * rng.random(n))
        if kind == "sparse":
            m[rng.random(n) < 0.5] = 0.0
        if kind == "front":
            m[n // 3:] = 0.0
        m[rng.integers(max(1, n // 3))] = 1.0
    return m.astype(np.float32)


@pytest.mark.parametrize("kind", ["flat", "peaked", "sparse", "front"])
@pytest.mark.parametrize("n,unit", [(1, 1), (32, 1), (100, 1), (256, 1), (2500, 1), (4096, 1), (16, 4), (592, 4), (4748, 4)])
def test_draw_is_one_element_with_mass(model, n, unit, kind):
    rng = np.random.Generator(np.random.Philox(1000 * n + unit))
    top = [np.float32(1.0 - j * 2.0 ** -24) for j in range(1, 17)]
    for _ in range(40):
        m = masses(rng, n, kind)
        c = np.cumsum(m.astype(np.float64))
        edges = np.float32(c[rng.integers(n, size=64)] / c[-1])
        for u in [np.float32(0.0), *top, *edges[edges < 1.0], *rng.random(8, dtype=np.float32)]:
            at, rest = model(m, unit, u)
            assert 0 <= at < n and m[at] > 0, (at, float(u))
            before = c[at - 1] if at else 0.0
            assert before - EPS * c[-1] <= float(u) * c[-1] < c[at] + EPS * c[-1], (at, float(u))
            assert abs(rest - (float(u) * c[-1] - before)) <= EPS * c[-1]


def test_nothing_to_draw_from(model):
    assert model(np.zeros(100, np.float32), 1, 0.5)[0] == -1
    assert model(np.full(100, np.nan, np.float32), 1, 0.5)[0] == -1
