"""Outlier-split weights on more than 256 super-blocks of rows x 32 columns: builds of one column per wave (two columns took up to 1.4
times as long there), several batches per wave, K that cuts one, sparse parts from empty to full: the bytes of the dense descriptor."""
import re

import pytest

from tests.gpu_util import kernels_of

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frac", [0.0, 0.01, 0.1, 1.0])
@pytest.mark.parametrize("kernel,build,M,N,K,a_off", [
    ("skinny16", (1, 4, 4, 1), 7, 8230, 1100, 0), ("skinny16", (1, 4, 4, 1), 40, 2900, 4163, 3), ("skinny16", (1, 4, 4, 1), 33, 2752, 2176, 5),
    ("skinny16", (1, 4, 2, 1), 50, 4300, 1100, 0), ("skinny16", (1, 4, 2, 1), 130, 1900, 4163, 3), ("skinny16", (1, 4, 2, 1), 97, 2350, 300, 5),
    ("skinny16", (1, 16, 4, 2), 32, 4096, 2560, 0), ("skinny16", (1, 8, 4, 2), 32, 4070, 2300, 0),   # 256: not yet
    ("skinny16", (1, 8, 4, 1), 9, 200, 6144, 0), ("skinny16", (1, 8, 4, 1), 20, 70, 4163, 1), ("skinny16", (1, 16, 4, 1), 9, 200, 6200, 0),
    ("skinny32", (2, 4, 2, 1), 65, 2900, 1030, 0), ("skinny32", (2, 4, 2, 1), 8, 8240, 130, 1), ("skinny32", (2, 4, 2, 1), 97, 2080, 4163, 2),
    ("skinny32", (2, 8, 4, 2), 64, 4096, 1100, 0),
    ("skinny64", (4, 4, 2, 1), 65, 4300, 500, 0), ("skinny64", (4, 4, 2, 1), 130, 2750, 130, 3), ("skinny64", (4, 8, 2, 2), 65, 4300, 530, 0),
    # batches of two end where a wave would have more offsets than lanes
    ("skinny16", (1, 4, 2, 1), 300, 864, 16384, 0), ("skinny16", (1, 4, 4, 1), 300, 864, 16400, 0),
    ("skinny32", (2, 4, 2, 1), 300, 830, 16384, 0), ("skinny32", (2, 8, 4, 2), 300, 830, 16400, 0),
])
def test_many_blocks(frac, kernel, build, M, N, K, a_off):
    import torch
    from paper_2101_05615_amd import qgemm as q
    g = torch.Generator(device="cuda").manual_seed(M * 7 + K)
    print(f"outlier blocks {M}x{N}x{K} frac {frac} {kernel}", flush=True)
    B = torch.randint(-8, 8, (K, N), dtype=torch.int8, device="cuda", generator=g)
    big = torch.rand((K, N), device="cuda", generator=g) < frac
    B = torch.where(big, torch.randint(8, 128, (K, N), dtype=torch.int8, device="cuda", generator=g), B)
    A = torch.randint(0, 256, (M, K + 16), dtype=torch.uint8, device="cuda", generator=g)[:, a_off:a_off + K]
    zp = torch.randint(-8, 9, (N,), generator=torch.Generator().manual_seed(1)).numpy()
    scales = torch.full((N,), 2.0 ** -12, device="cuda")
    split, dense = q.pack_b_outlier(B, zp), q.pack_b(B, zp)
    out = torch.empty((M, N), dtype=torch.uint8, device="cuda")
    (name,) = kernels_of(lambda: q.gemm_u8s8_requant(A, 130, split, None, scales, 100, False, out=out, kernel=kernel))
    m = re.search(r"qg_gemm_skinny_kernelILi0ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELb1E", name)
    assert m and tuple(int(x) for x in m.groups()) == build, name
    got = q.gemm_u8s8_requant(A, 130, split, None, scales, 100, False, kernel=kernel)
    want = q.gemm_u8s8_requant(A, 130, dense, None, scales, 100, False, kernel="tile64")
    assert torch.equal(got, want)
    x, rs = q.gemm_u8s8_acc32(A, split, want_rowsum=True, kernel=kernel)
    assert torch.equal(x, (A.double() @ B.double()).to(torch.int32)) and torch.equal(rs, A.to(torch.int32).sum(1, dtype=torch.int32))
