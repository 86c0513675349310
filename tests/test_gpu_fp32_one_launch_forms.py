"""fp32 activations with a workspace in one launch: the quantized rows that it leaves there, from every build that the automatic choice
takes for it (16, 32 and 64 rows, one and two columns per wave, two batches per wave, ragged M, N and K).  The recorded kernel is
compared, so that a new choice cannot leave a build without its test; that a call runs one launch is the same assertion."""
import re

import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import kernels_of, say

pytestmark = pytest.mark.gpu


# rows / 16, waves, k blocks per batch, columns; batches of a wave
@pytest.mark.parametrize("build,batches,M,N,K", [
    ((1, 4, 4, 1), 1, 18, 13, 109), ((1, 4, 4, 1), 1, 183, 98, 1024), ((1, 4, 4, 1), 1, 512, 15, 275),
    ((1, 8, 4, 1), 1, 5, 14, 1061), ((1, 8, 4, 1), 1, 511, 15, 1069),
    ((1, 8, 4, 2), 1, 2, 5075, 1375), ((1, 8, 4, 2), 1, 439, 146, 1088), ((1, 8, 4, 2), 1, 30, 2190, 2048),
    ((1, 8, 4, 2), 2, 2, 4124, 2390), ((1, 8, 4, 2), 2, 3, 4300, 2325), ((1, 8, 4, 2), 2, 1, 4447, 2228),   # copied between batches
    ((1, 16, 4, 1), 1, 1, 2375, 3828), ((1, 16, 4, 1), 1, 2, 3457, 4093),
    ((2, 8, 4, 1), 1, 17, 3738, 397), ((2, 8, 4, 1), 1, 476, 227, 478),
    ((2, 8, 4, 2), 1, 20, 7860, 1533), ((2, 8, 4, 2), 1, 21, 6741, 60), ((2, 8, 4, 2), 1, 512, 293, 101),
    ((4, 8, 2, 2), 1, 35, 4405, 1005), ((4, 8, 2, 2), 1, 50, 6477, 31), ((4, 8, 2, 2), 1, 512, 551, 484),
], ids=str)
def test_copy_of_every_build(build, batches, M, N, K):
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"fp32 one launch {build} {M} {N} {K}")
    case = wl.random_gemm(M + N + K, M, N, K)
    gen = torch.Generator(device="cuda").manual_seed(M + K)
    F = (torch.randn(M * (K + 3) + 8, device="cuda", generator=gen) * 3)[1:1 + M * (K + 3)].view(M, K + 3)[:, :K]
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    bias, scales = torch.from_numpy(case.bias).cuda(), torch.from_numpy(case.scales).cuda()
    ldq = K + (-K) % 16
    Aq = torch.full((M, ldq), 0xEE, dtype=torch.uint8, device="cuda")
    Aq[:, :K] = q.quantize_a_f32(F, 0.02, case.a_zp)
    blocks = -(-K // 64)
    assert -(-(-(-blocks // build[1])) // build[2]) == batches
    for fn, last in ((q.gemm_f32s8_requant, (case.c_zp, case.relu)), (q.gemm_f32s8_dequant_f32, (case.relu,))):
        results = []
        for kernel in ("auto", "tile64"):
            ws = torch.full((M * ldq + 64,), 0xEE, dtype=torch.uint8, device="cuda")
            names = kernels_of(lambda: fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=ws, kernel=kernel))
            if kernel == "auto":
                # <mode, row blocks, waves, batch, columns, 4-bit, source, ...>; source 1: fp32 rows
                m = re.search(r"qg_gemm_skinny_kernelILi\dELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb0ELi1E", names[0])
                assert len(names) == 1 and m and tuple(int(v) for v in m.groups()) == build, names
            results.append(fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=ws, kernel=kernel))
            assert torch.equal(ws[:M * ldq].view(M, ldq), Aq) and bool((ws[M * ldq:] == 0xEE).all()), kernel
        assert torch.equal(*results)


# without a workspace, by id: 64 rows from 17 k blocks on and 16 rows from 96 on run on sixteen waves
@pytest.mark.parametrize("build,M,N,K", [
    ((4, 8, 2, 1), 42, 300, 1024), ((4, 16, 2, 1), 42, 300, 1025), ((4, 16, 2, 1), 64, 70, 2048), ((4, 16, 2, 1), 61, 49, 2111),
    ((4, 16, 2, 1), 130, 500, 4099), ((4, 16, 2, 1), 33, 13, 7168), ((4, 8, 2, 2), 64, 4128, 1088),
    ((1, 8, 4, 1), 16, 48, 6080), ((1, 16, 4, 1), 16, 48, 6081), ((1, 16, 4, 1), 10, 43, 8192), ((1, 16, 4, 1), 117, 64, 7683),
    ((1, 8, 4, 2), 16, 4128, 6144), ((1, 4, 4, 1), 3, 4128, 6144),
], ids=str)
def test_sixteen_waves(build, M, N, K):
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"fp32 by id {build} {M} {N} {K}")
    case = wl.random_gemm(M + N + K, M, N, K)
    F = (torch.randn(M * (K + 1) + 8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(K)) * 3)[3:3 + M * (K + 1)].view(M, K + 1)[:, :K]
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    bias, scales = torch.from_numpy(case.bias).cuda(), torch.from_numpy(case.scales).cuda()
    kernel = f"skinny{16 * build[0]}"
    for fn, last in ((q.gemm_f32s8_requant, (case.c_zp, case.relu)), (q.gemm_f32s8_dequant_f32, (case.relu,))):
        (name,) = kernels_of(lambda: fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=q.NO_WORKSPACE, kernel=kernel))
        m = re.search(r"qg_gemm_skinny_kernelILi\dELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb0ELi1E", name)
        assert m and tuple(int(v) for v in m.groups()) == build, name
        got = fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=q.NO_WORKSPACE, kernel=kernel)
        assert torch.equal(got, fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, kernel="tile64"))


# without a workspace, the choice left to the library: us on the kernel of the queries, on this one
@pytest.mark.parametrize("M,N,K,rows", [(39, 2393, 1792, 16),    # 11.3, 6.4
                                        (78, 1603, 3264, 16),    # 18.7, 10.1
                                        (68, 1967, 1054, 32),    # 9.6, 6.1
                                        (16, 4096, 4096, 16)])
def test_choice_without_a_workspace(M, N, K, rows):
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"fp32 without a workspace {M} {N} {K}")
    case = wl.random_gemm(M + N + K, M, N, K)
    F = torch.randn((M, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(K)) * 3
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    scales = torch.from_numpy(case.scales).cuda()
    for fn, last in ((q.gemm_f32s8_requant, (case.c_zp, case.relu)), (q.gemm_f32s8_dequant_f32, (case.relu,))):
        (name,) = kernels_of(lambda: fn(F, 0.02, case.a_zp, Bp, None, scales, *last, workspace=q.NO_WORKSPACE))
        m = re.search(r"qg_gemm_skinny_kernelILi\dELi(\d+)E", name)
        assert m and 16 * int(m.group(1)) == rows, name
        assert torch.equal(fn(F, 0.02, case.a_zp, Bp, None, scales, *last, workspace=q.NO_WORKSPACE), fn(F, 0.02, case.a_zp, Bp, None, scales, *last, kernel="tile64"))
