"""The kernel of an automatic call on outlier-split weights: no call needs more than the queries announce, and calls without a workspace
run the kernel that is the fastest as the kernels are now, not as they were when the constants of the queries were fitted."""
import ctypes
import re

import pytest

from test_automatic_choice import descriptor


def split_descriptor(K, N, share):
    d = descriptor(K, N)
    d.split, d.frag_ptr, d.entries, d.nnz = 1, 4096, 4096, int(share * K * N)
    return d


def test_no_call_needs_more_than_was_announced():
    import torch
    if torch.cuda.is_available():
        pytest.skip("the calls that pass their checks would be launched")
    from paper_2101_05615_amd import qgemm as q
    split = 0
    for M in [1, 2, 16, 17, 33, 64, 65, 300, 1000, 5748]:
        for N in [16, 42, 64, 103, 256, 1024, 4096, 8192]:
            for K in [17, 128, 255, 768, 2048, 4097, 8192, 16384, 32768]:
                for share in (0.0, 0.005, 0.1):
                    h = ctypes.byref(split_descriptor(K, N, share))
                    p, dq = q.RequantParams(0, None, 4096, 1, 0, 0), q.DequantParams(0, None, 4096, 1, 0)
                    need = q.lib.qg_gemm_workspace_bytes(M, h)
                    split += need > 0
                    for a, lda, c, ldc in ((4096, K + (-K) % 16, 4096, N + (-N) % 16), (4097, K + 1, 4096, N)):
                        for rc in (q.lib.qg_gemm_u8s8_requant_splitk(a, M, lda, h, ctypes.byref(p), c, ldc, 4096, 0, None, 0, 0),
                                   q.lib.qg_gemm_u8s8_acc32_splitk(a, M, lda, h, 4096, ldc, None, 4096, 0, None, 0, 0)):
                            assert rc == (q.EWORKSPACE if need else q.ELAUNCH), (M, N, K, share, a, need, rc)
                        rc = q.lib.qg_gemm_u8s8_dequant_f32(a, M, lda, h, ctypes.byref(dq), 4096, ldc, 4097, None, 0)
                        assert rc == (q.EALIGN if need else q.ELAUNCH), (M, N, K, share, a, need, rc)
                        # a split that the caller asks for: as the queries say
                        want = q.lib.qg_gemm_splitk_workspace_bytes(M, h, 0, 3)
                        rc = q.lib.qg_gemm_u8s8_requant_splitk(a, M, lda, h, ctypes.byref(p), c, ldc, 4096, max(want, 16) - 16, None, 0, 3)
                        assert rc == (q.EWORKSPACE if want else q.ELAUNCH), (M, N, K, share, a, want, rc)
    assert split > 50


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,share,rows", [
    # us on the kernel that was chosen, on this one
    (89, 4784, 1408, 0.005, 32),     # 10.2, 6.5
    (22, 5040, 768, 0.001, 16),      # 4.3, 3.6
    (19, 6576, 640, 0.01, 16),       # 4.4, 3.7
    (132, 11392, 384, 0.05, 32),     # 13.9, 10.9
    (16, 8192, 8192, 0.005, 16),
    (1, 4096, 4096, 0.005, 16),
])
def test_kernel_of_the_call(M, N, K, share, rows):
    import torch
    from paper_2101_05615_amd import qgemm as q
    from gpu_util import kernels_of, say
    say(f"split choice {M} {N} {K} {share}")
    g = torch.Generator(device="cuda").manual_seed(M + N)
    B = torch.randint(-8, 8, (K, N), dtype=torch.int8, device="cuda", generator=g)
    B[torch.rand((K, N), device="cuda", generator=g) < share] = 77
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, device="cuda", generator=g)
    Bp, scales = q.pack_b_outlier(B, [0]), torch.full((1,), 2.0 ** -10, device="cuda")
    (name,) = kernels_of(lambda: q.gemm_u8s8_requant(A, 128, Bp, None, scales, 100, False))
    m = re.search(r"qg_gemm_skinny_kernelILi0ELi(\d+)E", name)
    assert m and 16 * int(m.group(1)) == rows, name
    want = q.gemm_u8s8_requant(A, 128, Bp, None, scales, 100, False, kernel="skinny64")
    ws = q.gemm_workspace(M, Bp)
    for w in (None, ws):
        assert torch.equal(q.gemm_u8s8_requant(A, 128, Bp, None, scales, 100, False, workspace=w), want)
    assert torch.equal(q.gemm_u8s8_acc32(A, Bp), q.gemm_u8s8_acc32(A, Bp, kernel="skinny64"))
