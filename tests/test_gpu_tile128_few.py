"""The 128 x 64 form of the 128-row kernel (at most one tile per CU, four wave sets that split K): numbers of k tiles that
leave none to four of them over (the last one ragged), rows and columns that end inside the tile, unaligned rows, every
output mode, against the CPU oracle: identical bytes.  The largest shape of the form and the smallest of the other one."""
import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, dev_case, oracle_gemm, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [768, 832, 896, 960, 1024, 1000, 1023, 1090, 2047])
@pytest.mark.parametrize("M,N,lda_pad,a_off", [(128, 64, 0, 0), (1, 40, 0, 0), (200, 130, 16, 0), (300, 200, 5, 3)])
def test_tile128_few_tiles(K, M, N, lda_pad, a_off):
    import torch
    from paper_2101_05615_amd import qgemm as q
    import oracle
    oracle.build()
    dev = torch.device("cuda:0")
    case = wl.random_gemm(K + M, M, N, K)
    say(f"tile128 few {M}x{N}x{K} lda+{lda_pad} offset {a_off}")
    A, B, bias, scales, C, c_store = dev_case(case, torch, dev, lda_pad=lda_pad, a_off=a_off)
    for zp in (True, False):   # with and without the row sums in the loop
        if not zp:
            case.b_zp[:] = 0
        Bp = q.pack_b(B, case.b_zp)
        q.gemm_u8s8_requant(A, case.a_zp, Bp, bias, scales, case.c_zp, case.relu, out=C, kernel="tile128")
        torch.cuda.synchronize()
        assert_same(C.cpu().numpy(), oracle_gemm(case, oracle), f"tile128 {M}x{N}x{K} theta_B {zp}")
    x, rs = q.gemm_u8s8_acc32(A, Bp, want_rowsum=True, kernel="tile128")
    f = q.gemm_u8s8_dequant_f32(A, case.a_zp, Bp, bias, scales, False, kernel="tile128")
    f64 = q.gemm_u8s8_dequant_f32(A, case.a_zp, Bp, bias, scales, False, kernel="tile64")
    torch.cuda.synchronize()
    assert_same(x.cpu().numpy(), case.A.astype(np.int32) @ case.B.astype(np.int32), f"acc32 {M}x{N}x{K}")
    assert_same(rs.cpu().numpy(), case.A.astype(np.int32).sum(1), f"row sums {M}x{N}x{K}")
    assert_same(f.cpu().numpy(), f64.cpu().numpy(), f"fp32 {M}x{N}x{K}")


@pytest.mark.parametrize("M,N,K", [(1024, 2048, 768), (1025, 2048, 768)])
def test_tile128_forms_meet(M, N, K):
    import torch
    from paper_2101_05615_amd import qgemm as q
    g = torch.Generator(device="cuda").manual_seed(3)
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, device="cuda", generator=g)
    B = torch.randint(-128, 128, (K, N), dtype=torch.int8, device="cuda", generator=g)
    Bp = q.pack_b(B, [0])
    got = q.gemm_u8s8_acc32(A, Bp, kernel="tile128")
    want = (A.double() @ B.double()).to(torch.int32)
    assert torch.equal(got, want), f"tile128 {M}x{N}x{K}"


@pytest.mark.parametrize("a_off,lda_pad", [(0, 0), (1, 0), (0, 3), (2, 2)])
def test_automatic_choice_with_a_split(a_off, lda_pad):
    """An automatic kernel with a K split asked for, on a shape whose automatic kernel without one is the 128 x 64 form."""
    import torch
    from paper_2101_05615_amd import qgemm as q
    M, N, K = 141, 6144, 4096
    assert q.kernel_names()[q.kernel_select(M, N, K)] == "tile128"
    say(f"auto + split {M}x{N}x{K} offset {a_off} lda+{lda_pad}")
    case = wl.random_gemm(7, M, N, K)
    A, B, bias, scales, C, c_store = dev_case(case, torch, torch.device("cuda:0"), lda_pad=lda_pad, a_off=a_off)
    Bp = q.pack_b(B, case.b_zp)
    want = q.gemm_u8s8_requant(A, case.a_zp, Bp, bias, scales, case.c_zp, case.relu, kernel="tile64")
    plain = q.gemm_u8s8_requant(A, case.a_zp, Bp, bias, scales, case.c_zp, case.relu, workspace=q.gemm_workspace(M, Bp))
    assert torch.equal(plain, want)
    for ksplit in (2, 4):
        assert q.gemm_splitk_factor(M, Bp, ksplit=ksplit) == ksplit
        ws = q.gemm_workspace(M, Bp, ksplit=ksplit)
        got = q.gemm_u8s8_requant_splitk(A, case.a_zp, Bp, bias, scales, case.c_zp, case.relu, ws, ksplit=ksplit)
        torch.cuda.synchronize()
        assert torch.equal(got, want), ksplit


def test_fp32_activations_without_a_workspace():
    import torch
    from paper_2101_05615_amd import qgemm as q
    M, N, K = 129, 6144, 4096
    assert q.kernel_names()[q.kernel_select(M, N, K)] == "tile128"
    g = torch.Generator(device="cuda").manual_seed(9)
    A = torch.randn((M, K), device="cuda", generator=g)
    Bp = q.pack_b(torch.randint(-128, 128, (K, N), dtype=torch.int8, device="cuda", generator=g), [3])
    bias = torch.randint(-1000, 1001, (N,), dtype=torch.int32, device="cuda", generator=g)
    scales = torch.full((1,), 2.0 ** -13, device="cuda")
    for fn, last in ((q.gemm_f32s8_requant, (100, False)), (q.gemm_f32s8_dequant_f32, (False,))):
        want = fn(A, 25.0, 120, Bp, bias, scales, *last)
        got = fn(A, 25.0, 120, Bp, bias, scales, *last, workspace=q.NO_WORKSPACE)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
