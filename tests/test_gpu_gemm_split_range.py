"""Large FP32 products over the whole range of FP32: operands are split into
BF16 terms exactly at any scale, and values that the split does not reach run
on the FP32 matrix cores."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _ones_to_two(g, *shape):
    """Full-significand values, each part of magnitude [1, 2)."""
    def part():
        x = 1 + torch.rand(*shape, device="cuda:0", generator=g)
        return torch.where(torch.rand(*shape, device="cuda:0", generator=g) < 0.5, x, -x)
    return torch.complex(part(), part())


def _gemm(A, B, C0, ta, tb, al=1.0, be=0.0, tile=-1):
    from paper_2503_23144_amd import lrcc
    C = C0.clone()
    lrcc.gemm_set_tile(tile)
    try:
        lrcc.gemm(A, B, C, transa=bool(ta), transb=bool(tb), alpha=al, beta=be, noalloc=True)
        torch.cuda.synchronize()
    finally:
        lrcc.gemm_set_tile(-1)
    return C


@pytest.mark.parametrize("ea,eb", [(-60, 0), (-100, 20), (-112, 30), (-126, 30), (30, -126), (28, 28), (-126, -10)])
@pytest.mark.parametrize("ta,tb", [(0, 0), (1, 1)])
def test_products_scale_by_powers_of_two(ta, tb, ea, eb):
    """Every step of the product, the 3M sums among them, is unchanged by
    powers of two while its results are normal numbers (the subnormal 3M sums
    of operands at 2^-126 are exact): equal bits."""
    m, n, k = 2040, 2048, 2001
    print(f"scaled operands 2^{ea} 2^{eb} ta={ta} tb={tb}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(3)
    A, B = _ones_to_two(g, *((k, m) if ta else (m, k))), _ones_to_two(g, *((n, k) if tb else (k, n)))
    C0 = torch.zeros(m, n, dtype=torch.complex64, device="cuda:0")
    ref = _gemm(A, B, C0, ta, tb)
    got = _gemm(A * 2.0 ** ea, B * 2.0 ** eb, C0, ta, tb)
    want = ref.to(torch.complex128) * 2.0 ** (ea + eb)
    # an output below the normal numbers, or each of its at most eight partials, is
    # rounded once more: half the smallest number
    tol = 8 * 2.0 ** -150 if ea + eb < -100 else 0.0
    d = got.to(torch.complex128) - want
    assert max(float(d.real.abs().max()), float(d.imag.abs().max())) <= tol


def test_values_beyond_the_split_match_the_fp32_kernel():
    """Infinities, NaN, magnitudes of 2^32 and more, alone and beside small
    ones: the bits of the FP32 kernel (one chain of K, the same tile)."""
    m, n, k = 4096, 2048, 1100
    g = torch.Generator(device="cuda:0").manual_seed(4)
    A0, B0 = _ones_to_two(g, m, k), _ones_to_two(g, k, n)
    C0 = torch.zeros(m, n, dtype=torch.complex64, device="cuda:0")

    def edit(X, *entries):
        Y = X.clone()
        for i, j, v in entries:
            Y[i, j] = v
        return Y

    inf, nan = float("inf"), float("nan")
    cases = {
        "infinity in A": (edit(A0, (5, 7, complex(inf, 0))), B0),
        "infinities in B": (A0, edit(B0, (0, 3, complex(-inf, 1)), (9, 4, complex(2, inf)))),
        "NaN": (edit(A0, (4095, 1099, complex(1, nan))), B0),
        "rounds up to infinity in BF16": (edit(0 * A0, (0, 0, 3.4e38)), edit(0 * B0, (0, 0, 0.5))),
        "at the bound": (edit(A0, (17, 18, 2.0 ** 32)), B0),
        "large and small": (edit(1e-36 * A0, (1, 2, 1e38), (3, 4, 1e30)), edit(B0, (2, 0, 0), (4, 0, 1e-38))),
        "all large": (1e18 * A0, 1e15 * B0),
        "overflow": (1e20 * A0, 1e20 * B0),
    }
    for name, (A, B) in cases.items():
        print(name, flush=True)
        got, ref = (torch.view_as_real(_gemm(A, B, C0, 0, 0, tile=t)).cpu().numpy() for t in (-1, 0))
        assert np.array_equal(got, ref, equal_nan=True), name


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(2040, 2048, 2001), (6005, 1400, 3100), (2300, 5000, 6200)])
def test_large_values_in_split_and_blocked_products(ta, tb, m, n, k):
    """Chains of K side by side and one after the other, operands in row
    blocks, alpha and beta.  One large element in the last row and depth, so
    that it shows only in the last block.  The bound of the other GEMM tests,
    row by row."""
    print(f"large values m={m} n={n} k={k} ta={ta} tb={tb}", flush=True)
    g = torch.Generator(device="cuda:0").manual_seed(m + n + k)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex64, device="cuda:0", generator=g)  # noqa: E731
    A, B, C0 = rand(*((k, m) if ta else (m, k))), rand(*((n, k) if tb else (k, n))), rand(m, n)
    A[-1, -1] = 2.0 ** 40
    al, be = 0.6 - 0.2j, -0.3 + 0.7j
    got = _gemm(A, B, C0, ta, tb, al, be)
    D = torch.complex128
    ref = al * ((A.T if ta else A).to(D) @ (B.T if tb else B).to(D)) + be * C0.to(D)
    size = (A.abs().amax(0 if ta else 1)).double() * 5.0
    err = ((got.to(D) - ref).abs().amax(1) / size)
    assert float(err.max()) <= 20 * 2e-7 * k


@pytest.mark.parametrize("o,v,nb", [(9, 53, 20), (17, 37, 18)])
def test_products_of_large_vectors(o, v, nb):
    """Operands read through index maps, replayed from a graph that was
    captured with small vectors: a Jacobian product is linear, so vectors 2^40
    times larger give the same numbers within the bound of FP32 against FP64
    (2^-24 per rounding, sums of at most v^2 terms)."""
    from paper_2503_23144_amd import lrcc
    from paper_2503_23144_amd.synth import make_inputs
    print(f"large vectors o={o} v={v} nb={nb}", flush=True)
    inp = make_inputs(o, v, o + v, seed=o * v)
    c = lrcc.Context(precision="mixed", tol=1e-9)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    rng = np.random.default_rng(o + v)
    t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
    X = rng.standard_normal((nb, c.n)) + 1j * rng.standard_normal((nb, c.n))
    c.sigma("residual", t)
    c.set_amplitudes(lrcc.AMP_T, t)
    for side in ("right", "left"):
        ref = c.sigma(side, X, precision="fp64")
        for e in (0, 0, 0, 40, 0, 40):
            got = c.sigma(side, X * 2.0 ** e, precision="mixed") * 2.0 ** -e
            for r in range(nb):
                assert np.abs(got[r] - ref[r]).max() <= 1e-5 * np.abs(ref[r]).max(), (side, e, r)
    c.close()
