"""GPU parity of the dense convolution over few input channels (image rows in LDS, a filter row of a pixel read as one
run of bytes) against the CPU oracle's direct convolution: identical bytes, nothing written outside the output."""
import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    dict(Nb=2, H=30, W=34, C=3, Cout=64, R=7, S=7, pad=3, stride=2),     # a first layer: two pieces per run, 7 steps
    dict(Nb=1, H=224, W=224, C=3, Cout=64, R=7, S=7, pad=3, stride=2),   # one tile cuts an image row
    dict(Nb=3, H=17, W=19, C=3, Cout=32, R=3, S=3, pad=1, stride=1),     # one 32-channel block, two steps, odd extents
    dict(Nb=2, H=9, W=300, C=4, Cout=20, R=3, S=3, pad=1, stride=2),     # output row cut into tiles, ragged Cout
    dict(Nb=1, H=12, W=13, C=1, Cout=16, R=5, S=5, pad=2, stride=1),     # run of 5 bytes: 3 steps, half a step of padding
    dict(Nb=1, H=1, W=3, C=3, Cout=7, R=3, S=3, pad=1, stride=1),        # 9 bytes of image: every chunk ends outside it
    dict(Nb=1, H=2, W=2, C=1, Cout=1, R=1, S=1, pad=0, stride=1),        # the smallest
    dict(Nb=2, H=6, W=5, C=24, Cout=40, R=3, S=3, pad=1, stride=1),      # five pieces per run, 8 steps
    dict(Nb=1, H=8, W=9, C=20, Cout=130, R=5, S=5, pad=2, stride=1),     # any number of steps, three column blocks
    dict(Nb=1, H=7, W=7, C=3, Cout=64, R=7, S=7, pad=6, stride=3),       # padding beyond the image on every side
    dict(Nb=1, H=10, W=11, C=5, Cout=33, R=2, S=4, pad=1, stride=2),     # even filter extents, K = 40
    dict(Nb=3, H=150, W=600, C=1, Cout=33, R=3, S=3, pad=1, stride=1),   # very many pixels: four waves holding the weights
    dict(Nb=2, H=6, W=5, C=7, Cout=24, R=1, S=1, pad=0, stride=1),       # 1 x 1: the gathering kernel
    dict(Nb=1, H=6, W=40, C=100, Cout=64, R=3, S=3, pad=1, stride=1),    # 29 steps: beyond this kernel, the gathering one
    # every number of steps with code of its own, and some without, in one and two column blocks
    dict(Nb=3, H=11, W=13, C=3, Cout=40, R=2, S=2, pad=1, stride=1),     # 1
    dict(Nb=2, H=14, W=11, C=2, Cout=48, R=7, S=7, pad=3, stride=1),     # 4
    dict(Nb=2, H=13, W=9, C=2, Cout=24, R=7, S=7, pad=3, stride=1),
    dict(Nb=2, H=9, W=10, C=5, Cout=40, R=5, S=5, pad=2, stride=1),      # 5
    dict(Nb=2, H=9, W=10, C=5, Cout=24, R=5, S=5, pad=2, stride=1),
    dict(Nb=2, H=9, W=10, C=11, Cout=72, R=4, S=4, pad=2, stride=1),     # 6; 72 channels: a column block of padding
    dict(Nb=2, H=13, W=9, C=3, Cout=24, R=7, S=7, pad=3, stride=1),      # 7
    dict(Nb=2, H=9, W=10, C=22, Cout=24, R=3, S=3, pad=1, stride=1),     # 8
    dict(Nb=2, H=20, W=130, C=33, Cout=64, R=3, S=3, pad=1, stride=8),   # the tile halved for the LDS
    dict(Nb=1, H=9, W=900, C=66, Cout=64, R=3, S=3, pad=1, stride=3),    # 77 KB of LDS
    dict(Nb=1, H=310, W=900, C=1, Cout=16, R=2, S=2, pad=0, stride=1),   # very many pixels, 1 and 3 steps
    dict(Nb=1, H=310, W=900, C=1, Cout=48, R=2, S=2, pad=0, stride=1),
    dict(Nb=1, H=310, W=900, C=3, Cout=24, R=5, S=5, pad=2, stride=1),
    dict(Nb=1, H=310, W=900, C=3, Cout=48, R=5, S=5, pad=2, stride=1),
    dict(Nb=2, H=60, W=60, C=4, Cout=16, R=5, S=5, pad=2, stride=2),     # words to gather, few pixels: the gathering kernel
])
@pytest.mark.parametrize("per_channel,with_bias,relu,c_zp,bzp", [
    (True, True, False, None, True), (False, False, True, 0, False), (True, True, True, 77, False), (True, False, False, 5, False)])
@pytest.mark.parametrize("offset", [0, 3])
def test_conv_few_channels_bit_exact(cfg, per_channel, with_bias, relu, c_zp, bzp, offset):
    import torch
    from paper_2101_05615_amd import qgemm as q
    import oracle
    oracle.build()
    dev = torch.device("cuda:0")
    say(f"conv runs {cfg} per_channel={per_channel} relu={relu} c_zp={c_zp} bzp={bzp} offset={offset}")
    c = wl.random_conv(21, G=1, per_channel=per_channel, with_bias=with_bias, relu=relu, **cfg)
    if c_zp is not None:
        c.c_zp = c_zp
    if not bzp:
        c.b_zp[:] = 0
    want = oracle.conv_groupwise_direct(c.inp, 1, c.wgt, c.a_zp, c.b_zp, c.bias, c.scales, c.c_zp, c.relu, c.pad, c.stride)
    Wp = q.pack_conv_dense_w(torch.from_numpy(np.ascontiguousarray(c.wgt[0])).to(dev), c.b_zp)
    store = torch.full((c.inp.size + 64,), 0xEE, dtype=torch.uint8, device=dev)
    inp = store[offset:offset + c.inp.size].view(c.inp.shape)
    inp.copy_(torch.from_numpy(c.inp).to(dev))
    res = torch.full((want.size + 64,), 0xEE, dtype=torch.uint8, device=dev)
    out = res[offset:offset + want.size].view(want.shape)
    bias = None if c.bias is None else torch.from_numpy(c.bias).to(dev)
    q.conv_dense_u8s8_requant(inp, Wp, c.a_zp, bias, torch.from_numpy(c.scales).to(dev), c.c_zp, c.relu, pad=c.pad,
                              stride=c.stride, out=out)
    torch.cuda.synchronize()
    assert_same(out.cpu().numpy(), want, f"conv {cfg}")
    rest = res.cpu().numpy()
    assert (rest[:offset] == 0xEE).all() and (rest[offset + want.size:] == 0xEE).all(), "bytes outside the output changed"
