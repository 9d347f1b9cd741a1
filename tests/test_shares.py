"""Which tiles the workgroups of a launch take, on the CPU: the library's own functions (csrc/shares.hpp) for every workgroup."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

HERE = Path(__file__).resolve().parent
CUS, XCDS = 256, 8
DEALT, CONTIGUOUS, EVEN = range(3)


@pytest.fixture(scope="module")
def share(tmp_path_factory):
    out = tmp_path_factory.mktemp("share") / "libshare_model.so"
    subprocess.run(["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-o", str(out), str(HERE / "share_model.cpp")], check=True)
    fn = ctypes.CDLL(str(out)).share_model
    fn.argtypes = [ctypes.c_int] * 6 + [ctypes.c_void_p]

    def tiles(T, groups, ksplit, unit, form, b):
        at = np.full(T, -1, np.int32)
        return at[:fn(T, groups, ksplit, unit, form, b, at.ctypes.data)]
    return tiles


def shapes():
    for ksplit in range(1, 9):
        most = CUS // ksplit
        for units in (1, 5, most - 1, most, most + 1, 2 * most + 7, 3 * most - 1, 10 * most, 17 * most + 9):
            for groups in {min(most, units), min(most, units, 5), min(most, units, 33)}:
                yield ksplit, groups, units


@pytest.mark.parametrize("unit", [1, 2])
@pytest.mark.parametrize("form", [DEALT, CONTIGUOUS, EVEN])
def test_every_tile_once_and_in_order(share, form, unit):
    """In order: of equal logits a lane keeps the one that it meets first, which has to be the lowest row."""
    for ksplit, groups, units in shapes():
        T = unit * units
        got = [share(T, groups, ksplit, unit, form, b) for b in range(groups)]
        assert np.array_equal(np.sort(np.concatenate(got)), np.arange(T))
        for t in got:
            assert (np.diff(t) > 0).all() and len(t) <= unit * -(-units // groups)
            assert (t.reshape(-1, unit) == t[::unit, None] + np.arange(unit)).all()


def test_an_xcd_reads_side_by_side(share):
    """In each whole round the workgroups of an XCD take one stretch.  Workgroup b of slice s is the launch's (s + ksplit b)th, and those go to
    the XCDs in turn."""
    for ksplit, groups, units in shapes():
        got = [share(units, groups, ksplit, 1, DEALT, b) for b in range(groups)]
        for s in range(ksplit):
            xcd = (s + ksplit * np.arange(groups)) % XCDS
            for u in range(units // groups):
                for x in set(xcd):
                    stretch = np.sort([got[b][u] for b in np.flatnonzero(xcd == x)])
                    assert (np.diff(stretch) == 1).all(), (ksplit, groups, units, u, x)
