"""The builds of the 64 x 128 patch kernel in which wave sets split K (64 x 64 tiles with four sets, 64 x 128 with two): slab
counts on both sides of the rule and off every multiple of the sets, slabs that hold two taps, K that ends mid-slab, tile counts
at one per CU and one more, ragged channel counts; with and without weight zero points; against the CPU oracle's direct
convolution: identical bytes."""
import dataclasses

import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    dict(Nb=2, H=9, W=7, C=64, Cout=64, R=3, S=3, pad=1),         # 9 slabs: one set
    dict(Nb=2, H=9, W=7, C=96, Cout=70, R=3, S=3, pad=1),         # 13.5 slabs: four sets of 4, 4, 3, 3, the last mid-slab
    dict(Nb=1, H=13, W=11, C=32, Cout=100, R=5, S=5, pad=2),      # 12.5 slabs of two taps each
    dict(Nb=3, H=7, W=7, C=160, Cout=33, R=3, S=3, pad=1),        # 22.5 slabs
    dict(Nb=1, H=6, W=5, C=64, Cout=17, R=5, S=5, pad=2),         # 25
    dict(Nb=1, H=1, W=1, C=256, Cout=1, R=3, S=3, pad=1),         # one pixel, one channel, 36
    dict(Nb=1, H=64, W=64, C=96, Cout=256, R=3, S=3, pad=1),      # 64 x 4 tiles: one per CU, four sets
    dict(Nb=1, H=65, W=64, C=160, Cout=256, R=3, S=3, pad=1),     # 65 x 4: too many; 65 x 2, two sets, 22.5 slabs
    dict(Nb=1, H=128, W=128, C=160, Cout=96, R=3, S=3, pad=1),    # 256 x 1, two sets
    dict(Nb=1, H=129, W=128, C=128, Cout=96, R=3, S=3, pad=1),    # 258 x 1: one set
])
@pytest.mark.parametrize("variant", range(3))
def test_patch_kernel_wave_sets(cfg, variant):
    import torch
    from paper_2101_05615_amd import qgemm as q
    import oracle
    oracle.build()
    dev = torch.device("cuda:0")
    say(f"conv patch sets {cfg} variant {variant}")
    c = wl.random_conv(41 + variant, G=1, relu=variant == 1, with_bias=variant != 2, **cfg)
    if variant == 0:
        c.b_zp[:] = 0
    c = dataclasses.replace(c, c_zp=[c.c_zp, 5, 0][variant])
    want = oracle.conv_groupwise_direct(c.inp, c.G, c.wgt, c.a_zp, c.b_zp, c.bias, c.scales, c.c_zp, c.relu, c.pad, c.stride)
    Wp = q.pack_conv_dense_w(torch.from_numpy(c.wgt[0]).contiguous().to(dev), c.b_zp)
    bias = None if c.bias is None else torch.from_numpy(c.bias).to(dev)
    for kernel in ("patch64x128", "auto"):
        got = q.conv_dense_u8s8_requant(torch.from_numpy(c.inp).to(dev), Wp, c.a_zp, bias, torch.from_numpy(c.scales).to(dev), c.c_zp,
                                        c.relu, pad=c.pad, stride=1, kernel=kernel)
        torch.cuda.synchronize()
        assert_same(got.cpu().numpy(), want, f"conv {cfg}, kernel {kernel}")
