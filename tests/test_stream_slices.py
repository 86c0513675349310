"""The order in which the streaming kernels deal slices of K to their waves, compiled for the host: within a workgroup every slice
once, and over the workgroups of one XCD (every eighth) a wave starts on all slices equally often where there are eight, on two where
there are sixteen.  All of them read all of A: with one order per XCD they ask for the same lines at the same time."""
import ctypes
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2101_05615_amd", "csrc")


@pytest.fixture(scope="module")
def slice_of(tmp_path_factory):
    d = tmp_path_factory.mktemp("slices")
    (d / "shim.cpp").write_text('#include "qg_stream.h"\nextern "C" int slice_of(int w, unsigned b, int n) { return qg_stream_slice(w, b, n); }\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(d / "shim.cpp"), "-o", str(d / "shim.so")], check=True)
    f = ctypes.CDLL(str(d / "shim.so")).slice_of
    f.argtypes = [ctypes.c_int, ctypes.c_uint, ctypes.c_int]
    return f


@pytest.mark.parametrize("waves", [4, 8, 16])
def test_every_slice_once_and_turned_within_an_xcd(slice_of, waves):
    for block in list(range(600)) + [2 ** 31 - 1, 2 ** 31, 2 ** 32 - 1]:
        assert sorted(slice_of(w, block, waves) for w in range(waves)) == list(range(waves)), block
    if waves != 8:   # (four waves: short K)
        assert all(slice_of(w, b, waves) == (w + b) % waves for w in range(waves) for b in range(600))
        assert waves == 4 or all(len({slice_of(0, xcd + 8 * j, waves) for j in range(8)}) == 2 for xcd in range(8))
        return
    for xcd in range(8):
        for wave in range(waves):
            starts = [slice_of(wave, xcd + 8 * j, waves) for j in range(2 * waves)]
            assert sorted(starts) == sorted(2 * list(range(waves))), (xcd, wave, starts)
        neighbours = [slice_of(0, 8 * xcd + j, waves) for j in range(8)]
        assert len(set(neighbours)) == min(waves, 8), neighbours
