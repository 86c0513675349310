"""Workgroup -> tile map of the 64 x 32 kernel: the tiles dealt to the XCDs one by one or in runs, whole and partial bands of
tile rows, numbers of tiles off every multiple of eight: every tile computed once, exact against 64-bit products."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tm,tn", [(35, 2), (19, 4), (18, 9), (10, 10), (33, 15),      # one by one
                                   (9, 1), (7, 19), (7, 7), (15, 13), (5, 20), (1, 9), (3, 3), (40, 12), (40, 13)])   # in runs
def test_every_tile_once(tm, tn):
    import torch
    from paper_2101_05615_amd import qgemm as q
    print(f"tile map {tm} x {tn}", flush=True)
    M, N, K = tm * 64 - 5, tn * 32 - 3, 200
    g = torch.Generator(device="cuda").manual_seed(tm * 100 + tn)
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, device="cuda", generator=g)
    B = torch.randint(-128, 128, (K, N), dtype=torch.int8, device="cuda", generator=g)
    Bp = q.pack_b(B, [0])
    x, rs = q.gemm_u8s8_acc32(A, Bp, want_rowsum=True, kernel="tile64x32k8")
    f = q.gemm_u8s8_dequant_f32(A, 0, Bp, None, torch.ones(1, device="cuda"), False, kernel="tile64x32k8")
    want = (A.double() @ B.double())
    torch.cuda.synchronize()
    assert torch.equal(x, want.to(torch.int32)) and torch.equal(rs, A.to(torch.int32).sum(1, dtype=torch.int32))
    assert torch.equal(f, want.float())
