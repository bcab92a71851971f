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
