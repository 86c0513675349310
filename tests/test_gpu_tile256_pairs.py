"""The 256 x 256 kernel's hand-scheduled loop requests A two 64-deep k tiles at a time: every small number of tiles (even
and odd, the shortest the loop takes, a ragged last tile behind it), rows that end inside either half of the tile, and row
starts off the cache lines, against the CPU oracle: identical bytes."""
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, dev_case, oracle_gemm, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [256, 320, 384, 448, 512, 576, 640, 703, 1090])
@pytest.mark.parametrize("M,N,lda_pad,a_off", [(256, 256, 0, 0), (1, 40, 0, 0), (129, 256, 16, 0), (600, 300, 5, 3)])
def test_tile256_every_tile_count(K, M, N, lda_pad, a_off):
    import torch
    from paper_2101_05615_amd import qgemm as q
    import oracle
    oracle.build()
    dev = torch.device("cuda:0")
    case = wl.random_gemm(K + M, M, N, K)
    say(f"tile256 pairs {M}x{N}x{K} lda+{lda_pad} offset {a_off}")
    A, B, bias, scales, C, c_store = dev_case(case, torch, dev, lda_pad=lda_pad, a_off=a_off)
    for zp in (True, False):   # with and without the row sums in the loop
        if not zp:
            case.b_zp[:] = 0
        Bp = q.pack_b(B, case.b_zp)
        q.gemm_u8s8_requant(A, case.a_zp, Bp, bias, scales, case.c_zp, case.relu, out=C, kernel="tile256")
        torch.cuda.synchronize()
        assert_same(C.cpu().numpy(), oracle_gemm(case, oracle), f"tile256 {M}x{N}x{K} theta_B {zp}")
