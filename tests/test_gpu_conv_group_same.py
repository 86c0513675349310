"""The stride-1 "same" kernel of the group convolution with square groups of 1 to 32 channels: images smaller than a wave's 32
pixels (several per wave, positions divided on the scalar unit), pixel counts and tile counts off every multiple, images so
wide that the channel slice is halved, grids large enough for the compact weights of groups of 1, 2 and 4 channels; with and
without weight zero points, against the CPU oracle's direct convolution: identical bytes."""
import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    dict(Nb=40, H=1, W=1, C=64, G=64),               # 3 x 3 on single pixels: every tap but the centre is outside
    dict(Nb=50, H=2, W=3, C=64, G=16),
    dict(Nb=3, H=5, W=31, C=96, G=96),               # 32-channel slices, three of them
    dict(Nb=2, H=33, W=17, C=128, G=64),             # groups of 2
    dict(Nb=1, H=129, W=1, C=128, G=16),             # one column, groups of 8; one pixel more than a tile
    dict(Nb=1, H=3, W=900, C=64, G=16),              # 64 channels of this row do not fit the LDS
    dict(Nb=1, H=3, W=900, C=64, G=4),
    dict(Nb=1, H=262, W=259, C=128, G=32),           # more than 1024 workgroups: compact weights, groups of 4
    dict(Nb=1, H=262, W=259, C=128, G=128),          # ... of 1
    dict(Nb=1, H=262, W=259, C=128, G=64),           # ... of 2
    dict(Nb=2, H=20, W=21, C=64, G=2),               # groups of 32
    dict(Nb=2, H=20, W=21, C=64, G=16, R=1, S=1, pad=0),
    dict(Nb=3, H=19, W=23, C=96, G=24, R=1, S=1, pad=0),        # 1 x 1, 32-channel slices: one chunk per thread
    dict(Nb=1, H=262, W=259, C=128, G=128, R=1, S=1, pad=0),    # 1 x 1, compact weights
    # wide rows and more workgroups than the CUs hold: the patch straight to LDS, in both channel slices
    dict(Nb=1, H=40, W=900, C=64, G=16),
    dict(Nb=1, H=40, W=900, C=64, G=64),
    dict(Nb=3, H=12, W=1021, C=96, G=12),
    dict(Nb=1, H=36, W=1064, C=64, G=4),                        # the widest that 64 channels fit
    dict(Nb=1, H=36, W=1065, C=64, G=4),
    dict(Nb=9, H=83, W=83, C=128, G=16),                        # fewer rounds of the grid without the gaps
])
@pytest.mark.parametrize("bzp,relu,c_zp", [(True, False, 77), (False, True, 0), (False, True, 9), (True, False, 0)])
def test_group_conv_same(cfg, bzp, relu, c_zp):
    import torch
    from paper_2101_05615_amd import qgemm as q
    import oracle
    oracle.build()
    dev = torch.device("cuda:0")
    say(f"group conv same {cfg} bzp={bzp} relu={relu} c_zp={c_zp}")
    c = wl.random_conv(31, relu=relu, **cfg)
    c.c_zp = c_zp
    if not bzp:
        c.b_zp[:] = 0
    want = oracle.conv_groupwise_direct(c.inp, c.G, c.wgt, c.a_zp, c.b_zp, c.bias, c.scales, c.c_zp, c.relu, c.pad, c.stride)
    Wp = q.pack_conv_w(torch.from_numpy(c.wgt).to(dev), c.b_zp)
    got = q.conv_groupwise_u8s8_requant(torch.from_numpy(c.inp).to(dev), Wp, c.a_zp, torch.from_numpy(c.bias).to(dev),
                                        torch.from_numpy(c.scales).to(dev), c.c_zp, c.relu, c.pad, c.stride)
    torch.cuda.synchronize()
    assert_same(got.cpu().numpy(), want, f"group conv {cfg}")


@pytest.mark.parametrize("H,W,R", [(1, 1 << 24, 1), (1 << 24, 1, 1), (1 << 24, 1, 3), (3, (1 << 23) + 5, 1)])
def test_group_conv_positions_of_long_images(H, W, R):
    """Rows and columns beyond 2^23 pixels: the last ones must not be taken for pixels outside the image.  A 1 x 1 filter
    does not know the shape of the image, and of a column of pixels a 3 x 3 filter sees the middle column only: the same
    pixels as an image of short rows, or the last ones as a shorter column, give the same bytes."""
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"group conv long image {H}x{W} filter {R}")
    g = torch.Generator(device="cuda").manual_seed(5)
    G, C, n = 8, 32, H * W
    wt = torch.randint(-128, 128, (G, R, R, 4, 4), dtype=torch.int8, device="cuda", generator=g)
    Wp = q.pack_conv_w(wt, np.zeros(1, np.int32))
    img = torch.randint(0, 256, (n, C), dtype=torch.uint8, device="cuda", generator=g)
    scales = torch.full((C,), 2.0 ** -7, device="cuda")
    bias = torch.zeros(C, dtype=torch.int32, device="cuda")
    got = q.conv_groupwise_u8s8_requant(img.view(1, H, W, C), Wp, 3, bias, scales, 100, False, R // 2, 1).view(n, C)
    if R == 1:
        side = 4096 if n == 1 << 24 else 3
        want = q.conv_groupwise_u8s8_requant(img.view(1, n // side, side, C), Wp, 3, bias, scales, 100, False, 0, 1).view(n, C)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
    else:
        for a, b in ((0, 5000), (n // 2, n // 2 + 5000), (n - 5000, n)):
            part = q.conv_groupwise_u8s8_requant(img[a:b].view(1, b - a, 1, C), Wp, 3, bias, scales, 100, False, 1, 1).view(b - a, C)
            torch.cuda.synchronize()
            lo, hi = (0 if a == 0 else 1), (b - a if b == n else b - a - 1)  # rows whose neighbours are all in the part
            assert torch.equal(got[a + lo:a + hi], part[lo:hi]), (a, b)
