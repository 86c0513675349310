"""Streaming kernels at the edges of their builds: the batches and the chunk that K cuts (from one byte on), rows at every
address, a quarter of a row block or less, the k-block counts at which the number of waves changes and the column counts at which
a wave takes two fragment columns; 8-bit, 4-bit and fp32 operands.  Whole numbers: every byte is the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2101_05615_amd import workloads as wl
from tests.gpu_util import assert_same, dev_case, say

pytestmark = pytest.mark.gpu

KS = [1, 15, 16, 17, 63, 65, 130, 1024, 1025, 1039, 2048, 2049, 4096, 4111, 4240]


@pytest.mark.parametrize("kernel", ["skinny16", "skinny32", "skinny64"])
@pytest.mark.parametrize("M,N", [(1, 40), (4, 4112), (5, 33), (8, 80), (9, 4100), (16, 2080), (33, 70), (64, 2090), (70, 300)])
def test_stream_ends(kernel, M, N):
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    for K in KS:
        if M * N * K > 3e8:
            continue
        a_off, lda_pad = [(0, 0), (0, -K % 16), (3, 5), (2, 6)][(K + M) % 4]
        say(f"stream ends {kernel} {M}x{N}x{K} off {a_off} lda +{lda_pad}")
        c = wl.unsaturated(wl.random_gemm(9000 + M + N + K, M, N, K, per_channel=True, with_bias=True, wide_zp=True))
        want = oracle.gemm_u8s8_requant(c.A, c.a_zp, c.B, c.b_zp, c.bias, c.scales, c.c_zp, c.relu)
        A, B, bias, scales, C, c_store = dev_case(c, torch, dev, lda_pad=lda_pad, a_off=a_off)
        q.gemm_u8s8_requant(A, c.a_zp, q.pack_b(B, c.b_zp), bias, scales, c.c_zp, c.relu, out=C, kernel=kernel)
        torch.cuda.synchronize()
        assert_same(C.cpu().numpy(), want, "8-bit weights")
        C.fill_(0xEE)
        q.gemm_u8s8_requant(A, c.a_zp, q.pack_b_outlier(B, c.b_zp), bias, scales, c.c_zp, c.relu, out=C, kernel=kernel)
        torch.cuda.synchronize()
        assert_same(C.cpu().numpy(), want, "4-bit weights, dense outliers")
        assert (c_store.cpu().numpy()[M * N:] == 0xEE).all(), "bytes past C were written"


@pytest.mark.parametrize("kernel", ["skinny16", "skinny32", "skinny64"])
@pytest.mark.parametrize("M,N", [(1, 40), (4, 4112), (17, 33), (40, 2080), (64, 500)])
def test_stream_ends_fp32(kernel, M, N):
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    for K in KS:
        if M * N * K > 2e8:
            continue
        say(f"stream ends fp32 {kernel} {M}x{N}x{K}")
        zp = [0, 90, 255][K % 3]
        Af, inv = wl.random_fp32_activations(M + K, M, K, alpha=0.02, zp=zp)
        c = wl.unsaturated(wl.random_gemm(9100 + M + N + K, M, N, K, per_channel=True, with_bias=True, a_zp=zp, wide_zp=True))
        Aq = oracle.quantize_f32(Af, inv, zp)
        want = oracle.gemm_u8s8_dequant_f32(Aq, zp, c.B, c.b_zp, c.bias, c.scales, True)
        store = torch.full((M, K + K % 3), float("nan"), dtype=torch.float32, device=dev)
        store[:, :K] = torch.from_numpy(Af).to(dev)
        got = q.gemm_f32s8_dequant_f32(store[:, :K], inv, zp, q.pack_b(torch.from_numpy(c.B).to(dev), c.b_zp),
                                       torch.from_numpy(c.bias).to(dev), torch.from_numpy(c.scales).to(dev), True,
                                       workspace=q.NO_WORKSPACE, kernel=kernel)
        aq = q.quantize_a_f32(store[:, :K], inv, zp)
        torch.cuda.synchronize()
        assert_same(np.ascontiguousarray(got.cpu().numpy()).view(np.int32), np.ascontiguousarray(want).view(np.int32), "one launch")
        assert_same(aq.cpu().numpy(), Aq, "quantization pass")
