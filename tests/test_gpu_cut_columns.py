"""Columns that N cuts inside a 16-byte store: every remainder, at aligned and odd addresses of C, on the kernels that store 16 (tiles,
patch convolution) or 4 (streaming) columns of a row at a time.  Bytes are the oracle's, and none beside them is written."""
import pytest

import oracle
from paper_2101_05615_amd import workloads as wl
from tests.gpu_util import assert_same, dev_case, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["skinny16", "tile64k1", "tile64k4", "tile64x32k8", "tile128", "tile256"])
def test_cut_columns(kernel):
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    for rest in range(16):
        for ldc_pad, c_off in ((0, 0), ((-rest) % 16, 0), (3, 5)):
            M, N, K = 37, 80 + rest, 832
            say(f"cut columns {kernel} N {N} ldc +{ldc_pad} at {c_off}")
            c = wl.unsaturated(wl.random_gemm(7700 + rest, M, N, K, per_channel=True, with_bias=True, wide_zp=True))
            want = oracle.gemm_u8s8_requant(c.A, c.a_zp, c.B, c.b_zp, c.bias, c.scales, c.c_zp, c.relu)
            A, B, bias, scales, C, c_store = dev_case(c, torch, dev, ldc_pad=ldc_pad, c_off=c_off)
            q.gemm_u8s8_requant(A, c.a_zp, q.pack_b(B, c.b_zp), bias, scales, c.c_zp, c.relu, out=C, kernel=kernel)
            torch.cuda.synchronize()
            assert_same(C.cpu().numpy(), want, "requant")
            C.fill_(0xEE)
            assert (c_store.cpu().numpy() == 0xEE).all(), "bytes beside C were written"


@pytest.mark.parametrize("kernel", ["patch64x128", "patch128x64", "patch256"])
@pytest.mark.parametrize("cout", [33, 39, 44, 47, 62])
def test_cut_columns_of_a_patch_convolution(kernel, cout):
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    c = wl.random_conv(cout, Nb=2, H=9, W=11, C=64, G=1, Cout=cout)
    say(f"cut columns {kernel} Cout {cout}")
    want = oracle.conv_groupwise_direct(c.inp, c.G, c.wgt, c.a_zp, c.b_zp, c.bias, c.scales, c.c_zp, c.relu, c.pad, c.stride)
    Wp = q.pack_conv_dense_w(torch.from_numpy(c.wgt[0]).to(dev), c.b_zp)
    got = q.conv_dense_u8s8_requant(torch.from_numpy(c.inp).to(dev), Wp, c.a_zp, torch.from_numpy(c.bias).to(dev),
                                    torch.from_numpy(c.scales).to(dev), c.c_zp, c.relu, c.pad, c.stride, kernel=kernel)
    torch.cuda.synchronize()
    assert_same(got.cpu().numpy(), want, "conv")
