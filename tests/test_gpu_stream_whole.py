"""Streaming kernels where every wave of every slice of K has whole batches: the build without the code for a K that cuts one, whatever
the number of waves (chosen for sixteen alone, that is for slices 4096 deep, four and eight took up to a tenth more time)."""
import re

import pytest

import oracle
from paper_2101_05615_amd import workloads as wl
from tests.gpu_util import assert_same, dev_case, kernels_of, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,ksplit,waves,columns,whole", [
    (1, 40, 1024, 1, 4, 1, True), (16, 4128, 1024, 1, 4, 1, True), (13, 70, 1024, 1, 4, 1, True),
    (5, 300, 2048, 1, 8, 1, True), (16, 64, 4096, 1, 16, 1, True), (3, 4128, 2048, 1, 8, 2, True), (80, 1520, 2048, 1, 8, 2, True),
    (16, 4100, 4096, 1, 8, 2, True), (17, 2080, 6144, 1, 8, 2, True),
    (16, 48, 4096, 2, 8, 1, True), (7, 48, 4096, 4, 4, 1, True), (16, 48, 8192, 2, 16, 1, True),   # slices
    # four waves, batches of eight: K from 8192 on and 64 M weights and more, rows counted 16 at a time
    (5, 8192, 8192, 1, 4, 2, True), (16, 6580, 10240, 1, 4, 2, True), (130, 890, 16384, 1, 4, 2, True), (16, 4096, 16384, 2, 4, 2, True),
    (16, 8160, 8192, 1, 8, 2, True), (16, 8200, 8128, 1, 8, 2, False), (3, 8192, 8192, 1, 4, 1, False),
    (5, 300, 1023, 1, 4, 1, False), (5, 300, 1025, 1, 8, 1, False), (5, 300, 960, 1, 4, 1, False), (5, 300, 1088, 1, 8, 1, False),
    (16, 64, 8192, 1, 8, 1, False), (16, 4100, 4032, 1, 8, 2, False), (16, 48, 4032, 2, 8, 1, False), (7, 48, 4096, 3, 8, 1, False),
])
def test_whole_batches(M, N, K, ksplit, waves, columns, whole):
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    say(f"whole batches {M}x{N}x{K} in {ksplit}")
    c = wl.unsaturated(wl.random_gemm(9300 + M + N + K, M, N, K, per_channel=True, with_bias=True, wide_zp=True))
    want = oracle.gemm_u8s8_requant(c.A, c.a_zp, c.B, c.b_zp, c.bias, c.scales, c.c_zp, c.relu)
    A, B, bias, scales, C, c_store = dev_case(c, torch, dev, lda_pad=3, a_off=5)
    Bp = q.pack_b(B, c.b_zp)
    if ksplit == 1:
        def call():
            q.gemm_u8s8_requant(A, c.a_zp, Bp, bias, scales, c.c_zp, c.relu, out=C, kernel="skinny16")
    else:
        ws = q.gemm_workspace(M, Bp, kernel="skinny16", ksplit=ksplit)

        def call():
            q.gemm_u8s8_requant_splitk(A, c.a_zp, Bp, bias, scales, c.c_zp, c.relu, ws, out=C, kernel="skinny16", ksplit=ksplit)
    (name,) = kernels_of(call)
    # <mode, row blocks, waves, batch, columns, 4-bit, source, ahead, whole>
    m = re.search(r"qg_gemm_skinny_kernelILi0ELi1ELi(\d+)ELi([48])ELi(\d+)ELb0ELi0ELb([01])ELb([01])EE", name)
    assert m and (int(m.group(1)), int(m.group(3)), m.group(5) == "1") == (waves, columns, whole), name
    assert int(m.group(2)) == (8 if whole and (waves, columns) == (4, 2) else 4), name
    assert not whole or (m.group(4) == "1") == (waves == 8 and K // ksplit > 64 * 4 * waves), name   # one batch: none requested ahead
    for _ in range(2):
        C.fill_(0xEE)
        call()
        torch.cuda.synchronize()
        assert_same(C.cpu().numpy(), want, "requant")
