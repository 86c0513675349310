"""fp32 output of the tiled kernels, whose MFMA operands change places for it: edges of tiles in both directions, unaligned output
rows, and nothing written outside the rows.  Reference: the product in float64 on the CPU, exact for these operands."""
import pytest

pytestmark = pytest.mark.gpu

KERNELS = ["tile64k1", "tile64", "tile64k4", "tile64x32k8", "tile128", "tile128x256", "tile256"]


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("K", [64, 320, 777])
@pytest.mark.parametrize("M,N,pad", [(1, 1, 0), (31, 33, 3), (33, 31, 1), (127, 129, 0), (129, 127, 5), (255, 257, 2), (257, 255, 1), (256, 256, 0)])
def test_fp32_output_edges(kernel, K, M, N, pad):
    import torch
    from paper_2101_05615_amd import qgemm as q
    g = torch.Generator().manual_seed(M * 7 + N * 3 + K)
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, generator=g)
    B = torch.randint(-128, 128, (K, N), dtype=torch.int8, generator=g)
    bias = torch.randint(-1000, 1001, (N,), dtype=torch.int32, generator=g)
    scales = (2.0 ** torch.randint(-12, -8, (N,), generator=g)).float()
    for b_zp in (0, 3):
        Bp = q.pack_b(B.cuda(), [b_zp])
        store = torch.full((M + 2, N + pad), -7.0, device="cuda")
        out = store[1:M + 1, :N]
        q.gemm_u8s8_dequant_f32(A.cuda(), 100, Bp, bias.cuda(), scales.cuda(), False, out=out, kernel=kernel)
        # every integer here is below 2^24 times a power of two: the fp32 result is exact
        acc = (A.double() - 100) @ (B.double() - b_zp) + bias.double()
        assert float(acc.abs().max()) < 2 ** 24
        want = torch.full((M + 2, N + pad), -7.0)
        want[1:M + 1, :N] = (acc * scales.double()).float()
        torch.cuda.synchronize()
        assert torch.equal(store.cpu(), want), (kernel, M, N, K, pad, b_zp)


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("ldc", [(1 << 20) - 1, 1 << 20])
def test_rows_far_apart(kernel, ldc):
    """Output rows 4 MiB apart: the widest that 32-bit offsets inside a tile reach, and the first that go by 64-bit addresses."""
    import torch
    from paper_2101_05615_amd import qgemm as q
    M, N, K = 133, 70, 96
    g = torch.Generator().manual_seed(ldc)
    A = torch.randint(0, 256, (M, K), dtype=torch.uint8, generator=g)
    B = torch.randint(-128, 128, (K, N), dtype=torch.int8, generator=g)
    scales = torch.full((N,), 2.0 ** -10)
    Bp = q.pack_b(B.cuda(), [3])
    store = torch.full(((M + 1) * ldc,), -7.0, device="cuda")
    out = store[:M * ldc].view(M, ldc)[:, :N]
    q.gemm_u8s8_dequant_f32(A.cuda(), 100, Bp, None, scales.cuda(), False, out=out, kernel=kernel)
    want = (((A.double() - 100) @ (B.double() - 3)) * 2.0 ** -10).float()   # exact, as above
    torch.cuda.synchronize()
    assert torch.equal(out.cpu(), want)
    out.fill_(-7.0)
    assert bool((store == -7.0).all())   # nothing else was written
