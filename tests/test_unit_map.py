"""The order in which workgroups take the sparse kernels' work units (unit_map.h, built
here by the host compiler): every unit once, and for any number of (b, g) each XCD (of
eight, in turn) gets its part of the units that exist and of the heavy ones among
them, which stand first in each (b, g)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2601_02819_amd", "csrc")


@pytest.fixture(scope="module")
def unit_at(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("unit_map")
    (d / "m.cpp").write_text('#define PHSA_HD static inline\n#include "unit_map.h"\n'
                             'extern "C" int run(int R, int per, int *bg, int *idx) {\n'
                             '  for (int x = 0; x < R * per; ++x) {\n'
                             '    const phsa::UnitAt a = phsa::unit_at(x, R, per);\n'
                             '    if (a.u != a.bg * per + a.idx) return 1;\n'
                             '    bg[x] = a.bg;\n    idx[x] = a.idx;\n  }\n  return 0;\n}\n')
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "m.so"), str(d / "m.cpp")], check=True)
    f = ctypes.CDLL(str(d / "m.so")).run

    def at(R, per):
        bg, idx = np.empty(R * per, np.int32), np.empty(R * per, np.int32)
        assert not f(R, per, *(a.ctypes.data_as(ctypes.POINTER(ctypes.c_int)) for a in (bg, idx)))
        return bg, idx

    return at


@pytest.mark.parametrize("per", [8, 24, 168, 1024])
def test_every_unit_once_and_fair_shares(unit_at, per):
    for R in [*range(1, 42), 64, 96, 100, 255, 256]:
        bg, idx = unit_at(R, per)
        assert bg.min() >= 0 and bg.max() < R and idx.min() >= 0 and idx.max() < per
        assert np.unique(bg.astype(np.int64) * per + idx).size == R * per
        xcd = np.arange(R * per) % 8
        for share in (1.0, 0.5, 0.125):            # the first part of every (b, g)'s units
            n = np.bincount(xcd[idx < per * share], minlength=8)
            # a group's XCDs differ by at most one unit per (b, g) that they share
            assert n.max() - n.min() <= max(1, R), (R, per, share, n)
            assert per < 1000 or n.max() <= 1.1 * n.mean(), (R, per, share, n)
