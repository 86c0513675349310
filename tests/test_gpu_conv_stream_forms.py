"""The builds of the streaming convolution that need many pixels or a long K, through the automatic choice: two fragment columns per
wave, 32 rows, several batches of taps requested one ahead of the other, ragged pixels and output channels.  The recorded kernel is
compared too, so that a new choice cannot leave a build without its test."""
import re

import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import assert_same, kernels_of, say
from test_gpu_conv_dense import env, run, want  # noqa: F401

pytestmark = pytest.mark.gpu


# source (2: whole 64-channel slices, 3: any 16 channels), rows / 16, waves, k blocks per batch, columns; batches of a wave
@pytest.mark.parametrize("build,batches,cfg", [
    ((3, 1, 4, 4, 1), 1, dict(Nb=1, H=5, W=5, C=16, Cout=32, R=5, S=5, pad=2)),
    ((3, 1, 4, 4, 1), 1, dict(Nb=1, H=7, W=6, C=32, Cout=48, R=5, S=5, pad=2, stride=2)),
    ((3, 1, 4, 4, 1), 1, dict(Nb=1, H=9, W=4, C=16, Cout=16, R=4, S=8, pad=4)),
    ((3, 1, 8, 4, 2), 1, dict(Nb=5, H=11, W=23, C=48, Cout=40, R=5, S=5, pad=2)),
    ((3, 1, 8, 4, 2), 2, dict(Nb=24, H=6, W=14, C=240, Cout=40, pad=0)),
    ((3, 1, 8, 4, 2), 3, dict(Nb=11, H=10, W=20, C=240, Cout=24, R=5, S=5, pad=2)),
    ((3, 2, 8, 4, 2), 1, dict(Nb=6, H=18, W=20, C=80, Cout=40, R=4, S=4, pad=2)),
    ((3, 2, 4, 4, 2), 3, dict(Nb=1, H=18, W=35, C=240, Cout=200)),
    ((3, 2, 16, 2, 1), 3, dict(Nb=18, H=12, W=6, C=240, Cout=200, R=5, S=5, pad=2, stride=2)),
    ((3, 1, 16, 4, 1), 1, dict(Nb=1, H=5, W=5, C=240, Cout=32, stride=2)),
    ((3, 1, 8, 4, 1), 3, dict(Nb=2, H=9, W=5, C=240, Cout=24, R=5, S=5, pad=0, stride=2)),
    ((2, 1, 8, 4, 2), 2, dict(Nb=10, H=15, W=23, C=128, Cout=24, R=5, S=5, pad=0)),
    ((2, 2, 8, 4, 2), 1, dict(Nb=16, H=24, W=6, C=128, Cout=40)),
    ((2, 2, 4, 4, 2), 3, dict(Nb=14, H=11, W=16, C=128, Cout=200, R=5, S=5, pad=2, stride=2)),
], ids=str)
def test_forms(env, build, batches, cfg):  # noqa: F811
    q, torch, dev, oracle = env
    say(f"streaming convolution {build} {cfg}")
    c = wl.random_conv(sum(cfg.values()), G=1, per_channel=True, **cfg)
    c.b_zp = np.zeros(1, np.int32)
    Wp = q.pack_conv_dense_w(torch.from_numpy(np.ascontiguousarray(c.wgt[0])).to(dev), c.b_zp)
    x, scales = torch.from_numpy(c.inp).to(dev), torch.from_numpy(c.scales).to(dev)
    out = torch.empty(want(c, oracle).shape, dtype=torch.uint8, device=dev)
    (name,) = kernels_of(lambda: q.conv_dense_u8s8_requant(x, Wp, c.a_zp, None, scales, c.c_zp, c.relu, pad=c.pad, stride=c.stride, out=out))
    # <mode, row blocks, waves, batch, columns, 4-bit, source, ...>
    m = re.search(r"qg_gemm_skinny_kernelILi0ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb0ELi(\d)E", name)
    assert m and (int(m.group(5)),) + tuple(int(v) for v in m.groups()[:4]) == build, name
    blocks = -(-c.wgt[0].size // c.wgt.shape[-1] // 64)
    assert -(-(-(-blocks // build[2])) // build[3]) >= batches
    assert_same(run(c, q, torch, dev), want(c, oracle), "conv")
    c.b_zp = np.arange(out.shape[-1], dtype=np.int32) % 17 - 8
    assert_same(run(c, q, torch, dev), want(c, oracle), "conv, zero points")
