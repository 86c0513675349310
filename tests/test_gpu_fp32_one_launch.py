"""fp32 activations with a workspace, automatic kernel: one launch where that is estimated to be faster (the streaming kernels quantize
what they stage), the quantized rows left in the workspace as by the two launches."""
import ctypes

import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lda_pad,off", [(0, 0), (3, 1)])
@pytest.mark.parametrize("M,N,K", [(1, 8, 64), (1, 8, 67), (3, 40, 200), (16, 16, 1030), (17, 48, 128), (16, 520, 513), (33, 257, 384), (40, 96, 4099),
                                   (64, 1024, 1024), (65, 200, 130), (128, 2500, 700), (16, 4100, 2048), (200, 64, 255), (512, 32, 96)])
def test_same_bytes_and_the_copy(M, N, K, lda_pad, off):
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"fp32 one launch {M} {N} {K} {lda_pad} {off}")
    case = wl.random_gemm(M + N + K, M, N, K)
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    store = torch.randn(M * (K + lda_pad) + 8, device="cuda", generator=gen) * 3
    F = store[off:off + M * (K + lda_pad)].view(M, K + lda_pad)[:, :K]
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    bias, scales = torch.from_numpy(case.bias).cuda(), torch.from_numpy(case.scales).cuda()
    ldq = K + (-K) % 16
    assert q.gemm_f32_workspace_bytes(M, Bp) == M * ldq
    Aq = torch.full((M, ldq), 0xEE, dtype=torch.uint8, device="cuda")
    Aq[:, :K] = q.quantize_a_f32(F, 0.02, case.a_zp)
    for fn, last in ((q.gemm_f32s8_requant, (case.c_zp, case.relu)), (q.gemm_f32s8_dequant_f32, (case.relu,))):
        results = []
        for kernel in ("auto", "tile64"):
            ws = torch.full((M * ldq + 64,), 0xEE, dtype=torch.uint8, device="cuda")
            results.append(fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=ws, kernel=kernel))
            assert torch.equal(ws[:M * ldq].view(M, ldq), Aq) and bool((ws[M * ldq:] == 0xEE).all())
        assert torch.equal(*results)


def test_a_workspace_off_16_bytes_is_refused():
    import torch
    from paper_2101_05615_amd import qgemm as q
    case = wl.random_gemm(5, 16, 64, 128)
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    F, scales = torch.zeros((16, 128), device="cuda"), torch.from_numpy(case.scales).cuda()
    ws, out = torch.zeros(1 << 13, dtype=torch.uint8, device="cuda"), torch.empty((16, 64), device="cuda")
    p = q.DequantParams(0, None, scales.data_ptr(), scales.numel(), 0)
    rc = q.lib.qg_gemm_f32s8_dequant_f32(F.data_ptr(), 16, 128, 50.0, Bp.handle, ctypes.byref(p), out.data_ptr(), 64, ws.data_ptr() + 8, None, 0)
    assert rc == q.EALIGN
