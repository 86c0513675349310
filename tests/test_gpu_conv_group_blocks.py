"""32-channel blocks per workgroup of the group convolution: one, two and four with taps from memory (stride 2), one and two with the
patch in LDS (stride 1).  The edges of the rules, ragged pixel tiles, with and without a weight zero point, against the CPU
oracle's direct convolution."""
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, say
from test_gpu_conv_groups import env, run, want  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    dict(Nb=1, H=7, W=9, C=128, G=32),                     # one block, 20 pixels
    dict(Nb=2, H=129, W=63, C=64, G=64),                   # 4160 pixels, 33 tiles x 2 blocks: one
    dict(Nb=1, H=255, W=255, C=64, G=8),                   # 16384 pixels, 128 tiles x 2 blocks: one
    dict(Nb=1, H=257, W=255, C=64, G=16),                  # 129 tiles x 2 blocks: the first with two
    dict(Nb=1, H=255, W=257, C=96, G=24),                  # C off 64: one
    dict(Nb=3, H=65, W=65, C=384, G=384),                  # 26 tiles x 12 blocks: two
    dict(Nb=1, H=223, W=221, C=512, G=16),                 # 98 tiles x 16 blocks: four
    dict(Nb=1, H=219, W=219, C=512, G=128),                # 95 tiles x 16 blocks: two
    dict(Nb=1, H=223, W=251, C=512, G=64),                 # 111 tiles x 16 blocks: four
    dict(Nb=1, H=223, W=253, C=512, G=32),                 # 112 tiles, a multiple of eight: two
    dict(Nb=1, H=119, W=121, C=896, G=28),                 # 29 tiles x 28 blocks: two
    dict(Nb=1, H=121, W=121, C=896, G=224),                # 30 tiles x 28 blocks, at most one workgroup per CU with four: four
    dict(Nb=1, H=191, W=253, C=192, G=48),                 # 96 tiles x 6 blocks, tiles a multiple of four: one
    dict(Nb=1, H=191, W=257, C=192, G=48),                 # 97 tiles x 6 blocks: two
    dict(Nb=1, H=100, W=101, C=1024, G=256, R=1, S=1, pad=0),  # 1 x 1, 20 tiles x 32 blocks: one
    dict(Nb=1, H=140, W=140, C=1024, G=1024, R=1, S=1, pad=0),  # 1 x 1, 39 tiles x 32 blocks: two
    dict(Nb=1, H=150, W=141, C=1024, G=32, R=1, S=1, pad=0),   # 1 x 1, 42 tiles x 32 blocks: four
    # stride 1
    dict(Nb=3, H=7, W=7, C=128, G=32, stride=1),           # one
    dict(Nb=11, H=80, W=80, C=128, G=32, stride=1),        # compact weights: one (two next to it)
    dict(Nb=6, H=112, W=112, C=128, G=64, stride=1),       # compact weights: one
    dict(Nb=6, H=112, W=113, C=128, G=128, stride=1),      # the same
    dict(Nb=5, H=56, W=56, C=192, G=6, stride=1),          # groups of 32: one
    dict(Nb=9, H=83, W=83, C=128, G=8, stride=1),          # one
    dict(Nb=32, H=56, W=56, C=128, G=32, stride=1),        # compact weights, no zero point: two; with one: one
    dict(Nb=22, H=54, W=54, C=128, G=32, stride=1),        # whole fragments, no zero point: two; with one: one
    dict(Nb=2, H=9, W=746, C=64, G=32, stride=1),          # wide: one, where the patch of two fits as well
    dict(Nb=1, H=40, W=400, C=192, G=24, stride=1),        # patch straight to LDS: two, with a zero point one
])
@pytest.mark.parametrize("b_zp", [False, True])
def test_blocks(env, cfg, b_zp):  # noqa: F811
    q, torch, dev, oracle = env
    cfg = dict(dict(stride=2), **cfg)
    c = wl.random_conv(17, **cfg)
    if not b_zp:
        c.b_zp[:] = 0
    say(f"{cfg} b_zp {b_zp}")
    assert_same(run(c, q, torch, dev), want(c, oracle), str(cfg))
