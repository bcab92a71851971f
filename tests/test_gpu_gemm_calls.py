"""lrcc_gemm and lrcc_gemm_noalloc: the same kernels and the same split over K."""
import numpy as np
import pytest
import torch

from test_gpu_gemm_paths import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(16, 33, 767), (15, 1, 768), (7, 200, 1500), (300, 12, 2047), (3, 70, 4099),
                                   (130, 90, 1800), (33, 65, 2049), (500, 40, 9001)])
def test_both_calls_give_the_same_bits(dtype, ta, tb, m, n, k):
    """Narrow and few-tile products on either side of the depth from which
    both calls split K."""
    from paper_2503_23144_amd import lrcc
    g = torch.Generator(device="cuda:0").manual_seed(m + n + k)
    rand = lambda *s: torch.randn(*s, dtype=dtype, device="cuda:0", generator=g)  # noqa: E731
    A, B, C0 = rand(*((k, m) if ta else (m, k))), rand(*((n, k) if tb else (k, n))), rand(m, n)
    out = []
    for noalloc in (False, True):
        C = C0.clone()
        lrcc.gemm(A, B, C, transa=bool(ta), transb=bool(tb), alpha=0.7 - 0.3j, beta=0.25 + 0.5j, noalloc=noalloc)
        torch.cuda.synchronize()
        out.append(C.cpu().numpy())
    assert np.array_equal(*out)


@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (17, 15, 24), (16400, 3, 7), (5, 16385, 25), (530, 513, 33),
                                   (17, 16, 25), (16, 33, 767), (15, 1, 768), (3, 70, 4099), (1800, 16, 600),
                                   (257, 130, 300), (33, 65, 2049), (31, 32, 9001)])
def test_allocating_call_matches_host(dtype, ta, tb, m, n, k):
    """The few-tile shapes through lrcc_gemm."""
    _check(dtype, ta, tb, m, n, k, noalloc=False)


@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(12500, 12600, 1100), (8100, 8200, 3072), (9814, 374, 3986), (5000, 5000, 3000)])
def test_blocks_of_the_operands_match_64_bits(ta, tb, m, n, k):
    """Large FP32 products whose packed operands exceed the static scratch:
    blocks of either extent and of the depth.  No further from 64 bits, row by
    row, than the FP32 matrix cores."""
    from paper_2503_23144_amd import lrcc
    print(f"blocked product m={m} n={n} k={k} ta={ta} tb={tb}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(m + n + k)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex64, device="cuda:0", generator=g)  # noqa: E731
    A, B, C0 = rand(*((k, m) if ta else (m, k))), rand(*((n, k) if tb else (k, n))), rand(m, n)
    al, be = 0.6 - 0.2j, -0.3 + 0.7j
    D = torch.complex128
    ref = al * ((A.T if ta else A).to(D) @ (B.T if tb else B).to(D)) + be * C0.to(D)
    rel = []
    for tile in (-1, 0):
        C = C0.clone()
        lrcc.gemm_set_tile(tile)
        try:
            lrcc.gemm(A, B, C, transa=bool(ta), transb=bool(tb), alpha=al, beta=be, noalloc=True)
            torch.cuda.synchronize()
        finally:
            lrcc.gemm_set_tile(-1)
        rel.append(float(((C - ref).abs() ** 2).sum(1).div((ref.abs() ** 2).sum(1)).sqrt().max()))
    assert rel[0] <= 1.1 * rel[1], rel
