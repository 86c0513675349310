"""fp32 activations with a workspace and a result that lies over them: all of A is read before C is written, also on shapes that
otherwise take one launch."""
import pytest

from paper_2101_05615_amd import workloads as wl
from gpu_util import kernels_of, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K", [(16, 512, 512), (64, 1024, 1024), (33, 96, 256), (16, 2048, 768)])
@pytest.mark.parametrize("where", ["over", "first row of A is last of C", "behind"])
def test_result_over_the_activations(M, N, K, where):
    import torch
    from paper_2101_05615_amd import qgemm as q
    say(f"fp32 in place {M} {N} {K} {where}")
    case = wl.random_gemm(M + N + K, M, N, K)
    w = max(N, K)
    store = torch.empty((3 * M, w), device="cuda")
    first = M if where != "behind" else 2 * M
    A = store[first:first + M, :K]
    F = torch.randn((M, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(M + K)) * 3
    row = {"over": M, "first row of A is last of C": 1, "behind": M}[where]
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    bias, scales = torch.from_numpy(case.bias).cuda(), torch.from_numpy(case.scales).cuda()
    ws = torch.empty(q.gemm_f32_workspace_bytes(M, Bp), dtype=torch.uint8, device="cuda")
    for fn, last, out in ((q.gemm_f32s8_dequant_f32, (case.relu,), store[row:row + M, :N]),
                          (q.gemm_f32s8_requant, (case.c_zp, case.relu), store.view(torch.uint8)[row:row + M, 4 * w - N:])):
        A.copy_(F)
        want = fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=ws)
        assert len(kernels_of(lambda: fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, workspace=ws))) == 1, "not a shape of one launch"
        apart = where == "behind" or (out.dtype == torch.uint8 and out.data_ptr() + (M - 1) * 4 * w + N <= A.data_ptr())
        assert len(kernels_of(lambda: fn(A, 0.02, case.a_zp, Bp, bias, scales, *last, out=out, workspace=ws))) == (1 if apart else 2)
        fn(A, 0.02, case.a_zp, Bp, bias, scales, *last, out=out, workspace=ws)
        assert torch.equal(out, want)
