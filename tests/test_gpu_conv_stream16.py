"""The streaming convolution for channel counts off 64, through the automatic choice (few pixels, long K: 5.2 to 6.3 us on the tiled
kernels, 4.2 here), against the direct oracle.  A 64-byte block of K holds pieces of up to four taps there."""
import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, say
from test_gpu_conv_dense import env, run, want  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cfg", [
    dict(Nb=1, H=5, W=5, C=16, Cout=32, R=5, S=5, pad=2),                # four taps per block, K = 400: a quarter of the last one
    dict(Nb=1, H=7, W=6, C=32, Cout=48, R=5, S=5, pad=2, stride=2),      # two taps per block
    dict(Nb=2, H=5, W=7, C=48, Cout=40),                                 # three pieces per tap
    dict(Nb=1, H=6, W=5, C=80, Cout=33, R=5, S=3, pad=1),                # five pieces, rows of C off 4 bytes
    dict(Nb=3, H=7, W=12, C=96, Cout=32),                                # 252 pixels
    dict(Nb=2, H=12, W=12, C=96, Cout=128, stride=2),
    dict(Nb=1, H=4, W=4, C=240, Cout=64, R=5, S=5, pad=4),               # padding beyond the filter's reach, K = 6000
    dict(Nb=2, H=6, W=6, C=176, Cout=512, R=4, S=4, pad=0),              # two row blocks by 16 column blocks
    dict(Nb=1, H=9, W=4, C=16, Cout=16, R=4, S=8, pad=4),                # 32 taps: all validity bits
], ids=lambda c: "x".join(str(v) for v in c.values()))
@pytest.mark.parametrize("bzp", [False, True])
def test_channels_off_64(env, cfg, bzp):  # noqa: F811
    q, torch, dev, oracle = env
    say(f"conv of channels off 64 {cfg} {bzp}")
    c = wl.random_conv(sum(cfg.values()) + bzp, G=1, per_channel=bzp, **cfg)
    if not bzp:
        c.b_zp = np.zeros(1, np.int32)
    assert_same(run(c, q, torch, dev), want(c, oracle), "conv of channels off 64")
