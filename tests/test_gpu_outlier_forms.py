"""Outlier-split weights: sparse parts from empty to more than 64 entries per batch of k blocks (several rounds of the
scatter), extreme values, both wave counts of every row-block kernel (more than 256 workgroups, and too few k blocks for
sixteen waves), ragged K and rows off the 16-byte grid: the bytes of the dense descriptor, which the oracle pins."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frac", [0.0, 0.01, 0.3, 1.0])
@pytest.mark.parametrize("M,N,K,a_off", [(16, 4224, 4096, 0), (5, 96, 4096, 0), (33, 200, 640, 0), (64, 2200, 4160, 0),
                                         (17, 70, 1000, 3), (40, 4300, 300, 0)])
@pytest.mark.parametrize("kernel", ["skinny16", "skinny32", "skinny64"])
def test_outlier_forms(frac, M, N, K, a_off, kernel):
    import torch
    from paper_2101_05615_amd import qgemm as q
    g = torch.Generator(device="cuda").manual_seed(M * 7 + K)
    print(f"outlier forms {M}x{N}x{K} frac {frac} {kernel}", flush=True)
    B = torch.randint(-8, 8, (K, N), dtype=torch.int8, device="cuda", generator=g)
    big = torch.rand((K, N), device="cuda", generator=g) < frac
    B = torch.where(big, torch.randint(0, 2, (K, N), dtype=torch.int8, device="cuda", generator=g) * 127 - 128 +
                    torch.randint(0, 129, (K, N), dtype=torch.int16, device="cuda", generator=g).to(torch.int8), B)
    A = torch.randint(0, 256, (M, K + 16), dtype=torch.uint8, device="cuda", generator=g)[:, a_off:a_off + K]
    zp = torch.randint(-8, 9, (N,), generator=torch.Generator().manual_seed(1)).numpy()
    scales = torch.full((N,), 2.0 ** -12, device="cuda")
    bias = torch.randint(-1000, 1001, (N,), dtype=torch.int32, device="cuda", generator=g)
    split, dense = q.pack_b_outlier(B, zp), q.pack_b(B, zp)
    assert split.nnz == int(((B < -8) | (B > 7)).sum())
    got = q.gemm_u8s8_requant(A, 130, split, bias, scales, 100, False, kernel=kernel)
    want = q.gemm_u8s8_requant(A, 130, dense, bias, scales, 100, False, kernel="tile64")
    x, rs = q.gemm_u8s8_acc32(A, split, want_rowsum=True, kernel=kernel)
    exact = (A.double() @ B.double()).to(torch.int32)
    torch.cuda.synchronize()
    assert torch.equal(got, want)
    assert torch.equal(x, exact) and torch.equal(rs, A.to(torch.int32).sum(1, dtype=torch.int32))
