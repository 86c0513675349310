"""QG_KERNEL_AUTO by the closer prices: no call needs more than the queries announce, whatever the alignment of its operands,
and the choice gives the bytes of a fixed kernel on the shapes where it turns from one kernel to another."""
import ctypes

import pytest

from paper_2101_05615_amd import workloads as wl
from test_automatic_choice import descriptor

MS = [1, 2, 16, 17, 33, 48, 64, 65, 129, 300, 1000, 5748, 25284]
NS = [16, 42, 64, 103, 256, 1024, 1531, 4096, 6304, 8192]
KS = [17, 32, 128, 255, 256, 767, 768, 1216, 2048, 2816, 4096, 4097, 8192, 16384, 65536]


def test_no_call_needs_more_than_was_announced():
    import torch
    if torch.cuda.is_available():
        pytest.skip("the calls that pass their checks would be launched")
    from paper_2101_05615_amd import qgemm as q
    split = 0
    for M in MS:
        for N in NS:
            for K in KS:
                h = ctypes.byref(descriptor(K, N))
                p, dq = q.RequantParams(0, None, 4096, 1, 0, 0), q.DequantParams(0, None, 4096, 1, 0)
                need = q.lib.qg_gemm_workspace_bytes(M, h)
                split += need > 0
                for a, lda, c, ldc in ((4096, K, 4096, N), (4096, K + (-K) % 16, 4096, N + (-N) % 16), (4100, K, 4097, N), (4097, K + 1, 4096, N)):
                    # a workspace of no bytes: refused exactly where the query asks for some
                    for rc in (q.lib.qg_gemm_u8s8_requant_splitk(a, M, lda, h, ctypes.byref(p), c, ldc, 4096, 0, None, 0, 0),
                               q.lib.qg_gemm_u8s8_acc32_splitk(a, M, lda, h, 4096, ldc, None, 4096, 0, None, 0, 0)):
                        assert rc == (q.EWORKSPACE if need else q.ELAUNCH), (M, N, K, a, lda, need, rc)
                    # a workspace that cannot be used, where nothing uses one
                    rc = q.lib.qg_gemm_u8s8_dequant_f32(a, M, lda, h, ctypes.byref(dq), 4096, ldc, 4097, None, 0)
                    assert rc == (q.EALIGN if need else q.ELAUNCH), (M, N, K, a, lda, need, rc)
    assert split > 50


def test_kernel_select_answers_for_whole_steps():
    from paper_2101_05615_amd import qgemm as q
    for M in MS:
        for N in NS:
            for K in KS[:-1]:
                assert q.kernel_select(M, N, K) == q.kernel_select(M, -(-N // 16) * 16, -(-K // 64) * 64), (M, N, K)


@pytest.mark.parametrize("M,N,K,fast", [
    # us with the kernel that an earlier fit chose, with the fastest
    (7, 6304, 2816, ("skinny16",)),                          # 6.4 on the 64 x 32 tile, 5.3
    (69, 3616, 2048, ("tile64x32k8",)),                      # 9.6, 6.2
    (827, 17, 15685, ("skinny16",)),                         # 25.1, 10.4: tall, few columns, long K
    (1152, 32, 11840, ("skinny16",)),                        # 18.7, 8.7
    (940, 64, 14177, ("skinny16",)),                         # 29.4, 16.1
    (1340, 11, 3072, ("skinny16",)),                         # 7.5, 5.1
    (64, 64, 128, ("tile64k1",)),                            # 3.5, 3.2
    (9, 7996, 5824, ("skinny16",)),                          # 10.1 on the 64 x 32 tile, 9.2
    (39460, 865, 87, ("tile128",)),                          # 26.9, 22.3 (rows of A and C off 16 bytes; the choice is the same)
    (80, 3072, 2048, ("skinny16",)),                         # 6.1, 4.8: rounds of the few-fat-waves form
    (96, 2048, 2048, ("skinny32", "skinny16")),              # 5.3, 4.6
    (640, 128, 8192, ("skinny16",)),                         # 9.7, 8.2
    (320, 768, 8192, ("skinny32",)),                         # 12.7, 10.2
    (2048, 128, 4096, ("tile64x32k8", "skinny32")),          # 9.8, 8.0 on both
    (12288, 384, 2048, ("tile128",)),                        # 21.3, 17.5: the last column of 256 half full
    (32768, 4096, 256, ("tile128x256",)),                    # 82.8, 69.9
    # 5 to 16 rows and more than 4096 columns: tiles had been chosen there
    (9, 6208, 6752, ("skinny16",)),                          # 10.9, 8.9
    (14, 5632, 3648, ("skinny16",)),                         # 7.1, 5.8
    (5, 7680, 3536, ("skinny16",)),                          # 8.2, 6.6
    (5, 6016, 4096, ("skinny16",)),                          # 7.5, 6.1
    (15, 4800, 4096, ("skinny16",)),                         # 6.5, 5.5
    (5, 6208, 6752, ("skinny16",)),
    (8, 16384, 2048, ("skinny16",)),                         # 7.8, 7.1
    (16, 14336, 4096, ("skinny16",)),                        # 11.2, 10.6
    (4, 14336, 4096, ("skinny16",)),                         # 11.0, 10.1
    (16, 11008, 4096, ("skinny16", "tile64k4")),             # 9.4 and 9.5
    (16, 28672, 4096, ("tile64", "tile128")),                # 20.2 and 20.5, 24.4 on the 16-row kernel
    (16, 8192, 8192, ("skinny16",)),                         # 12.9, 12.6
    # a long K and weights beyond the caches
    (16, 8192, 16384, ("skinny16",)),                        # 26.6 on the 64 x 64 tile with four sets, 25.2
    (8, 7168, 18432, ("skinny16",)),                         # 25.7, 24.8
    (16, 6144, 24576, ("skinny16",)),                        # 33.9, 30.6
    (16, 8192, 10240, ("skinny16",)),                        # 19.0, 17.5
])
def test_shapes_that_were_slow(M, N, K, fast):
    from paper_2101_05615_amd import qgemm as q
    assert q.kernel_names()[q.kernel_select(M, N, K)] in fast


def test_autotune_times_the_choice_of_the_call(monkeypatch):
    """The reported loss is that of an "auto" call, not of the kernel that kernel_select names."""
    from paper_2101_05615_amd import autotune, qgemm as q
    asked = []

    def timed(q_, torch_, M, N, K, kernels, *a):
        asked.append(list(kernels))
        return {k: 9.0 if k == "auto" else 10.0 + i if k != "tile64" else 6.0 for i, k in enumerate(kernels)}

    monkeypatch.setattr(autotune, "time_shape", timed)
    rows = autotune.tune(q, None, [(4, 16, 17)], log=lambda s: None)
    assert "auto" in asked[0] and rows[0]["best"] == "tile64" and rows[0]["auto_us"] == 9.0 and "auto" not in rows[0]["us"]
    assert rows[0]["auto"] == q.kernel_names()[q.kernel_select(4, 16, 17)]
    assert "1.5000x" in autotune.summary(rows) and autotune.table_from_rows(rows) == [[4, 4, 16, 16, 17, 17, "tile64"]]


@pytest.mark.gpu
@pytest.mark.parametrize("a_off,lda_pad", [(0, 0), (4, 4), (1, 3)])
@pytest.mark.parametrize("M,N,K", [(2, 6683, 2336), (6, 4996, 7488), (7, 6304, 2816), (49, 4938, 2048), (16, 42, 17), (63, 103, 255),
                                   (300, 520, 256), (129, 1531, 767), (1000, 200, 768), (5748, 256, 316), (2600, 1100, 2064), (64, 256, 16384)])
def test_choice_against_a_fixed_kernel(M, N, K, a_off, lda_pad):
    import torch
    from paper_2101_05615_amd import qgemm as q
    case = wl.random_gemm(M + N + K, M, N, K)
    lda = K + (-K) % 16 + lda_pad
    store = torch.zeros(M * lda + 32, dtype=torch.uint8, device="cuda")
    A = store[a_off:a_off + M * lda].view(M, lda)[:, :K]
    A.copy_(torch.from_numpy(case.A))
    Bp = q.pack_b(torch.from_numpy(case.B).cuda(), case.b_zp)
    bias, scales = torch.from_numpy(case.bias).cuda(), torch.from_numpy(case.scales).cuda()
    args = (A, case.a_zp, Bp, bias, scales)
    want = q.gemm_u8s8_requant(*args, case.c_zp, case.relu, kernel="tile64")
    ws = q.gemm_workspace(M, Bp)
    for w in (None, ws, torch.zeros(1 << 10, dtype=torch.uint8, device="cuda") if ws is None else ws):
        assert torch.equal(q.gemm_u8s8_requant(*args, case.c_zp, case.relu, workspace=w), want)
    assert torch.equal(q.gemm_u8s8_acc32(A, Bp), q.gemm_u8s8_acc32(A, Bp, kernel="tile64"))
    assert torch.equal(q.gemm_u8s8_dequant_f32(*args, case.relu), q.gemm_u8s8_dequant_f32(*args, case.relu, kernel="tile64"))
    F = torch.randn((M, K), device="cuda", generator=torch.Generator(device="cuda").manual_seed(5))
    for fn, last in ((q.gemm_f32s8_requant, (case.c_zp, case.relu)), (q.gemm_f32s8_dequant_f32, (case.relu,))):
        ref = fn(F, 0.02, case.a_zp, Bp, bias, scales, *last, kernel="tile64")
        assert torch.equal(fn(F, 0.02, case.a_zp, Bp, bias, scales, *last), ref)
    torch.cuda.synchronize()
