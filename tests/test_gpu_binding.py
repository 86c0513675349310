"""The extension module's calls against the ctypes path they stand in front of: the same bytes, outputs, workspaces and streams,
and for every argument that it does not take -- other types, failed checks, refused calls -- what the slow path does."""
import ctypes
import gc

import numpy as np
import pytest

from paper_2101_05615_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2101_05615_amd import qgemm as q
    dev = torch.device("cuda:0")
    c = wl.random_gemm(3, 70, 96, 200)
    t = dict(A=torch.from_numpy(c.A).to(dev), Bp=q.pack_b(torch.from_numpy(c.B).to(dev), c.b_zp), bias=torch.from_numpy(c.bias).to(dev),
             scales=torch.from_numpy(c.scales).to(dev))
    p = q._params(c.a_zp, t["bias"], t["scales"], c.c_zp, c.relu)
    want = torch.empty((70, 96), dtype=torch.uint8, device=dev)
    q._check(q.lib.qg_gemm_u8s8_requant(t["A"].data_ptr(), 70, 200, t["Bp"].handle, ctypes.byref(p), want.data_ptr(), 96, None, q._stream()), "")
    torch.cuda.synchronize()
    return q, torch, dev, c, t, want


def call(q, c, t, **over):
    a = dict(A=t["A"], a_zp=c.a_zp, Bp=t["Bp"], bias=t["bias"], scales=t["scales"], c_zp=c.c_zp, relu=c.relu)
    kw = {k: over.pop(k) for k in ("out", "workspace", "kernel") if k in over}
    a.update(over)
    return q.gemm_u8s8_requant(a["A"], a["a_zp"], a["Bp"], a["bias"], a["scales"], a["c_zp"], a["relu"], **kw)


def test_same_bytes_and_outputs(env):
    q, torch, dev, c, t, want = env
    assert q._binding.gemm_u8s8_requant(t["A"], c.a_zp, t["Bp"], t["bias"], t["scales"], c.c_zp, c.relu, None, None, 0) is not None
    for over in ({}, dict(kernel="tile64"), dict(kernel=q.kernel_id("skinny64")), dict(relu=int(c.relu)), dict(a_zp=np.int64(c.a_zp)),
                 dict(a_zp=float(c.a_zp)), dict(c_zp=torch.tensor(c.c_zp)), dict(workspace=torch.zeros(1 << 16, dtype=torch.uint8, device=dev))):
        got = call(q, c, t, **over)
        assert got.shape == (70, 96) and got.dtype == torch.uint8 and torch.equal(got, want), over
    wide = torch.full((70, 110), 9, dtype=torch.uint8, device=dev)
    out = wide[:, 3:99]
    assert call(q, c, t, out=out) is out and torch.equal(out, want) and bool((wide[:, :3] == 9).all()) and bool((wide[:, 99:] == 9).all())
    rows = torch.zeros((70, 333), dtype=torch.uint8, device=dev)
    rows[:, 5:205] = t["A"]
    assert torch.equal(call(q, c, t, A=rows[:, 5:205]), want)

    class Sub(torch.Tensor):
        pass
    assert torch.equal(call(q, c, t, A=t["A"].as_subclass(Sub)), want)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = call(q, c, t)
    s.synchronize()
    assert torch.equal(got, want)
    assert call(q, c, t, A=t["A"][:0]).shape == (0, 96)


def test_errors_are_those_of_the_checks(env):
    q, torch, dev, c, t, want = env
    for over in (dict(A=t["A"].int()), dict(A=t["A"].t()), dict(A=t["A"].cpu()), dict(A=t["A"][:, :199]), dict(scales=t["scales"].double()),
                 dict(bias=t["bias"].float()), dict(scales=t["scales"].repeat(2)[::2]), dict(out=torch.empty((70, 95), dtype=torch.uint8, device=dev)),
                 dict(out=torch.empty((70, 96), dtype=torch.int8, device=dev))):
        with pytest.raises(AssertionError):
            call(q, c, t, **over)
    for over, code in ((dict(a_zp=256), q.EINVAL), (dict(scales=t["scales"][:50]), q.EINVAL), (dict(kernel=99), q.EINVAL)):
        with pytest.raises(q.QGemmError) as e:
            call(q, c, t, **over)
        assert e.value.code == code
    with pytest.raises(ValueError):
        call(q, c, t, kernel="no such kernel")
    with pytest.raises(AttributeError):
        call(q, c, t, A=None)
    closed = q.pack_b(torch.zeros((200, 96), dtype=torch.int8, device=dev), [0])
    closed.close()
    with pytest.raises(AssertionError):
        call(q, c, t, Bp=closed)


def test_fp32_activations(env):
    q, torch, dev, c, t, _ = env
    A = torch.randn((70, 200), device=dev) * 2
    Aq = q.quantize_a_f32(A, 20.0, c.a_zp)
    want = q.gemm_u8s8_dequant_f32(Aq, c.a_zp, t["Bp"], t["bias"], t["scales"], True)
    ws = torch.empty(q.gemm_f32_workspace_bytes(70, t["Bp"]), dtype=torch.uint8, device=dev)
    out = torch.empty((70, 96), device=dev)
    for kw in ({}, dict(workspace=ws), dict(workspace=ws, out=out), dict(workspace=q.NO_WORKSPACE, kernel="skinny32"), dict(kernel="tile128")):
        got = q.gemm_f32s8_dequant_f32(A, 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], True, **kw)
        assert got.dtype == torch.float32 and torch.equal(got, want), kw
        assert ("out" in kw) == (got is out)
    want8 = call(q, c, t, A=Aq)
    assert torch.equal(q.gemm_f32s8_requant(A, np.float32(20.0), c.a_zp, t["Bp"], t["bias"], t["scales"], c.c_zp, c.relu), want8)
    # the module itself, not the path behind it: both outputs, own and given output and workspace
    for c_zp, ref in ((None, want), (c.c_zp, want8)):
        own = torch.zeros_like(ref)
        for o, w in ((None, None), (None, ws), (own, None), (own, ws)):
            relu = True if c_zp is None else c.relu
            got = q._binding.gemm_f32s8(A, 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], c_zp, relu, o, w, 0)
            assert got is not None and got.dtype == ref.dtype and torch.equal(got, ref), (c_zp, o is None, w is None)
            assert o is None or got is own
            own.zero_()
        for k in ("tile64", "skinny32"):
            got = q._binding.gemm_f32s8(A, 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], c_zp, relu, None, None, q.kernel_id(k))
            assert got is not None and torch.equal(got, ref), k
        assert q._binding.gemm_f32s8(A.double(), 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], c_zp, relu, None, None, 0) is None
    for bad in (0.0, float("nan")):
        with pytest.raises(q.QGemmError):
            q.gemm_f32s8_dequant_f32(A, bad, c.a_zp, t["Bp"], t["bias"], t["scales"], True)
    with pytest.raises(AssertionError):
        q.gemm_f32s8_dequant_f32(A.double(), 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], True)
    with pytest.raises(TypeError):
        q.gemm_f32s8_requant(A, 20.0, c.a_zp, t["Bp"], t["bias"], t["scales"], None, False)


def test_prepared_calls(env):
    q, torch, dev, c, t, want = env
    out = torch.zeros((70, 96), dtype=torch.uint8, device=dev)
    pg = q.PreparedGemm(t["A"].clone(), c.a_zp, t["Bp"], t["bias"].clone(), t["scales"].clone(), c.c_zp, c.relu, out)
    launch = pg.launch
    del pg
    gc.collect()
    junk = [torch.full((70, 200), 7, dtype=torch.uint8, device=dev) for _ in range(8)]   # would take the place of what was freed
    launch()
    torch.cuda.synchronize()
    assert torch.equal(out, want) and len(junk) == 8
    bad = q.PreparedGemm(t["A"], 300, t["Bp"], t["bias"], t["scales"], c.c_zp, c.relu, out)
    with pytest.raises(q.QGemmError) as e:
        bad.launch()
    assert e.value.code == q.EINVAL and "qg_gemm_u8s8_requant" in str(e.value)


def conv_operands(torch, c):
    bias = None if c.bias is None else torch.from_numpy(c.bias).cuda()
    return torch.from_numpy(c.inp).cuda(), bias, torch.from_numpy(c.scales).cuda()


@pytest.mark.parametrize("cfg", [dict(Nb=2, H=9, W=14, C=64, G=16, pad=1, stride=2), dict(Nb=3, H=12, W=7, C=64, G=64, pad=1, stride=1),
                                 dict(Nb=1, H=8, W=11, C=96, G=12, R=1, S=1, pad=0, stride=1)])
def test_prepared_group_convolution(env, cfg):
    q, torch, dev, *_ = env
    c = wl.random_conv(23, **cfg)
    x, bias, scales = conv_operands(torch, c)
    Wp = q.pack_conv_w(torch.from_numpy(c.wgt).cuda(), c.b_zp)
    want = q.conv_groupwise_u8s8_requant(x, Wp, c.a_zp, bias, scales, c.c_zp, c.relu, pad=c.pad, stride=c.stride)
    out = torch.zeros_like(want)
    q.PreparedConv(x, Wp, c.a_zp, bias, scales, c.c_zp, c.relu, c.pad, c.stride, out).launch()
    torch.cuda.synchronize()
    assert torch.equal(out, want)


@pytest.mark.parametrize("kernel", ["auto", "tile64", "patch128x64", "skinny16"])
@pytest.mark.parametrize("cfg", [dict(Nb=2, H=9, W=14, C=64, Cout=72, pad=1, stride=1), dict(Nb=2, H=9, W=14, C=64, Cout=72, R=3, S=2, pad=0, stride=2),
                                 dict(Nb=1, H=7, W=13, C=128, Cout=40, R=2, S=4, pad=1, stride=3)])
def test_prepared_dense_convolution(env, cfg, kernel):
    q, torch, dev, *_ = env
    c = wl.random_conv(29, G=1, **cfg)
    x, bias, scales = conv_operands(torch, c)
    Wp = q.pack_conv_dense_w(torch.from_numpy(np.ascontiguousarray(c.wgt[0])).cuda(), c.b_zp)
    want = q.conv_dense_u8s8_requant(x, Wp, c.a_zp, bias, scales, c.c_zp, c.relu, pad=c.pad, stride=c.stride, kernel="tile64k1")
    out = torch.zeros_like(want)
    call = q.PreparedConvDense(x, Wp, c.a_zp, bias, scales, c.c_zp, c.relu, c.pad, c.stride, out, kernel=kernel)
    if kernel.startswith("patch") and c.stride != 1:
        with pytest.raises(q.QGemmError) as e:   # (the kernel id arrived where it belongs)
            call.launch()
        assert e.value.code == q.EUNSUPPORTED and "qg_conv_dense_u8s8_requant" in str(e.value)
        return
    call.launch()
    torch.cuda.synchronize()
    assert torch.equal(out, want)
