"""QG_KERNEL_AUTO where the 128 x 64 form of the 128-row kernel is the choice for aligned rows: calls that ask for a K split
are accepted or refused alike for every alignment of A, and need what the queries announce.  Host logic: the descriptor is
made by hand, and every call fails its checks before anything is enqueued."""
import ctypes
import os
import re

import pytest

from paper_2101_05615_amd import qgemm as q

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Descriptor(ctypes.Structure):   # struct qg_packed_b
    _fields_ = [(n, ctypes.c_int) for n in ("kind", "version", "K", "N", "K_pad", "N_pad", "has_bzp", "n_b_zp")] + \
               [(n, ctypes.c_void_p) for n in ("packed", "col_off", "bzp")] + \
               [(n, ctypes.c_int) for n in ("G", "R", "S", "Cg", "Og")] + \
               [(n, ctypes.c_void_p) for n in ("conv_frags", "conv_any", "conv_gemm", "conv_gemm_off")] + \
               [(n, ctypes.c_int) for n in ("conv_gemm_kpad", "conv_gemm_npad", "split")] + \
               [("frag_ptr", ctypes.c_void_p), ("entries", ctypes.c_void_p), ("nnz", ctypes.c_longlong)]


def descriptor(K, N):
    text = open(os.path.join(ROOT, "paper_2101_05615_amd", "csrc", "qg_internal.h")).read()
    version = int(re.search(r"QG_LAYOUT_VERSION\s*=?\s*(\d+)", text).group(1))
    d = Descriptor(kind=1, version=version, K=K, N=N, K_pad=-(-K // 128) * 128, N_pad=-(-N // 256) * 256, packed=4096,
                   col_off=4096, bzp=4096)
    assert q.lib.qg_packed_b_k(ctypes.byref(d)) == K and q.lib.qg_packed_b_n(ctypes.byref(d)) == N
    return d


def few(M, N, K):   # at most one 128 x 64 tile per CU, K deep enough
    return -(-M // 128) * -(-N // 64) <= 256 and K >= 768 and q.kernel_names()[q.kernel_select(M, N, K)] == "tile128"


SHAPES = [(141, 6144, 4096), (129, 6144, 4096), (65, 12288, 2048), (80, 12288, 12288), (256, 8192, 8192), (999, 1531, 2047),
          (512, 4096, 2048), (128, 12288, 16384)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_explicit_split_does_not_depend_on_the_alignment(M, N, K):
    assert few(M, N, K), "not a shape of the form: choose another"
    d = descriptor(K, N)
    h = ctypes.byref(d)
    p = q.RequantParams(0, None, 4096, 1, 0, 0)
    for ksplit in (2, 3, 4, 8):
        factor = q.lib.qg_gemm_splitk_factor(M, h, 0, ksplit)
        need = q.lib.qg_gemm_splitk_workspace_bytes(M, h, 0, ksplit)
        assert (factor > 1) == (need > 0)
        for a, lda in ((4096, K + (-K) % 4), (4097, K + (-K) % 4), (4096, K + (-K) % 4 + 1), (4098, K + (-K) % 4 + 2)):
            # (one byte too few, so that an accepted split stops here; a kernel without one is refused)
            rc = q.lib.qg_gemm_u8s8_requant_splitk(a, M, lda, h, ctypes.byref(p), 4096, N, 4096, max(need, 16) - 16, None, 0, ksplit)
            assert rc == (q.EWORKSPACE if factor > 1 else q.EUNSUPPORTED), (ksplit, a, lda, rc)
            rc = q.lib.qg_gemm_u8s8_acc32_splitk(a, M, lda, h, 4096, N, None, 4096, max(need, 16) - 16, None, 0, ksplit)
            assert rc == (q.EWORKSPACE if factor > 1 else q.EUNSUPPORTED), (ksplit, a, lda, rc)


def test_no_split_by_itself_where_the_form_is_the_choice():
    """The form has no split, and what other rows run instead must not want one either: nothing was announced."""
    seen = 0
    for M in [65, 80, 97, 129, 141, 160, 200, 257, 385, 600, 999, 1024, 2000, 4096, 8192]:
        for N in [16, 64, 200, 512, 1024, 1531, 2048, 4096, 6144, 12288, 16384]:
            for K in [768, 1000, 2048, 4096, 8192, 16384, 32768]:
                if few(M, N, K):
                    seen += 1
                    d = descriptor(K, N)
                    assert q.lib.qg_gemm_splitk_factor(M, ctypes.byref(d), 0, 0) == 1, (M, N, K)
                    assert q.lib.qg_gemm_workspace_bytes(M, ctypes.byref(d)) == 0, (M, N, K)
    assert seen > 60


def test_fp32_activations_without_a_workspace():
    """The one-launch form on a streaming kernel stays the choice where that is the best kernel but for the form."""
    p, dq = q.RequantParams(0, None, 4096, 1, 0, 0), q.DequantParams(0, None, 4096, 1, 0)
    for M, N, K, one_launch in [(129, 6144, 4096, True), (141, 6144, 4096, True), (80, 12288, 12288, True), (65, 12288, 2048, True),
                                (256, 8192, 8192, False), (999, 1531, 2047, False)]:
        assert few(M, N, K)
        d = descriptor(K, N)
        # A off 4 bytes: the one-launch form refuses it, a tiled kernel refuses the missing workspace
        want = q.EALIGN if one_launch else q.EWORKSPACE
        assert q.lib.qg_gemm_f32s8_requant(4097, M, K, 1.0, ctypes.byref(d), ctypes.byref(p), 4096, N, None, None, 0) == want
        assert q.lib.qg_gemm_f32s8_dequant_f32(4097, M, K, 1.0, ctypes.byref(d), ctypes.byref(dq), 4096, N, None, None, 0) == want
