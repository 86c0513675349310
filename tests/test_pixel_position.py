"""Image positions of the stride-1 group convolution (row and column of a wave's lanes from exact divisions by invariants),
compiled for the host: extents up to 2^25, where fp32 quotients go wrong, and images smaller than a wave's 32 pixels."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2101_05615_amd", "csrc")

SHIM = r"""
#include "qg_position.h"
extern "C" long long bad_positions(unsigned W, unsigned H, unsigned begin, unsigned end) {
  const qg_udiv w = qg_make_udiv(W), h = qg_make_udiv(H);
  long long bad = 0;
  for (unsigned long long px = begin; px < end; ++px) {
    const unsigned first = (unsigned)px / 32 * 32;
    int row, col;
    qg_pixel_position(first, (unsigned)px - first, W, w.m, w.s, H, h.m, h.s, &row, &col);
    bad += row != (int)(px / W % H) || col != (int)(px % W);
  }
  return bad;
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("position")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.bad_positions.argtypes = [ctypes.c_uint] * 4
    lib.bad_positions.restype = ctypes.c_longlong
    return lib


@pytest.mark.parametrize("e", range(22, 26))
@pytest.mark.parametrize("d", [-1, 0, 1])
def test_long_rows_and_columns(shim, e, d):
    n = 2 ** e + d
    for W, H in ((n, 1), (1, n), (n // 3, 3), (3, n // 3), (31, n // 31), (32, n // 32), (33, n // 33)):
        total = W * H
        for begin in (0, total // 2, max(0, total - 4096)):
            assert shim.bad_positions(W, H, begin, min(begin + 4096, total)) == 0, (W, H, begin)
    assert shim.bad_positions(n, 1, 2 ** 31 - 2 ** 25, 2 ** 31 - 2 ** 25 + 100000) == 0   # many images of one row


def test_small_images(shim):
    for W in range(1, 70):
        for H in range(1, 40):
            assert shim.bad_positions(W, H, 0, 4000) == 0, (W, H)
            assert shim.bad_positions(W, H, 2 ** 26 - 1000, 2 ** 26) == 0, (W, H)
