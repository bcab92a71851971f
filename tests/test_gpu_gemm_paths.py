"""The complex GEMM's kernels at the edges of their tiles, steps and splits,
against the host product.  Operands sit in storage filled with NaN, so a
read or a write outside them shows in the result or in the guard."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _in_nan(x, dtype, pad=64):
    """x on the device inside a larger NaN-filled buffer: (view, buffer)."""
    buf = torch.full((x.size + 2 * pad,), complex("nan+nanj"), dtype=dtype, device="cuda:0")
    v = buf[pad:pad + x.size].view(x.shape)
    v.copy_(torch.tensor(x, dtype=dtype))
    return v, buf


def _check(dtype, ta, tb, m, n, k, noalloc):
    from paper_2503_23144_amd import lrcc
    rng = np.random.default_rng(m + 3 * n + 5 * k)
    rand = lambda *s: rng.standard_normal(s) + 1j * rng.standard_normal(s)  # noqa: E731
    A, B, C0 = rand(*((k, m) if ta else (m, k))), rand(*((n, k) if tb else (k, n))), rand(m, n)
    al, be = 0.6 - 0.2j, -0.3 + 0.7j
    ref = al * ((A.T if ta else A) @ (B.T if tb else B)) + be * C0
    Ad, _ = _in_nan(A, dtype)
    Bd, _ = _in_nan(B, dtype)
    Cd, buf = _in_nan(C0, dtype)
    lrcc.gemm(Ad, Bd, Cd, transa=bool(ta), transb=bool(tb), alpha=al, beta=be, noalloc=noalloc)
    torch.cuda.synchronize()
    got = Cd.cpu().numpy().astype(np.complex128)
    eps = 1e-15 if dtype == torch.complex128 else 2e-7
    scale = np.sqrt(k) * np.abs(A).max() * np.abs(B).max() + np.abs(C0).max()
    assert np.abs(got - ref).max() <= 20 * eps * scale * np.sqrt(k)
    assert torch.isnan(buf[:64].real).all() and torch.isnan(buf[-64:].real).all()


# shallow (k <= 24) on few and many tiles; one tile per wavefront (k <= 512, 1024
# tiles and more, narrow and wide); 16 x 16 tiles shared by 8 and 4 wavefronts, whole and
# split; 32 x 32 tiles, whole and split: each with remainders of the tile, the
# step (16 or 8 deep) and the wavefronts' round
@pytest.mark.parametrize("dtype", [torch.complex128, torch.complex64])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (17, 15, 24), (16400, 3, 7), (5, 16385, 25), (530, 513, 33),
                                   (17, 16, 25), (16, 33, 767), (15, 1, 768), (3, 70, 4099), (1800, 16, 600),
                                   (257, 130, 300), (33, 65, 2049), (31, 32, 9001)])
def test_gemm_few_tiles_matches_host(dtype, ta, tb, m, n, k):
    _check(dtype, ta, tb, m, n, k, noalloc=True)
