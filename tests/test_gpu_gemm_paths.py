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


# large FP32 products (operands split into three BF16 terms): both tiles, chains
# of K run side by side and one after the other, an operand packed in row blocks,
# remainders of every tile, slab and chain.  The bound is that of the other GEMM
# tests; inputs of mixed magnitude check that small rows keep their own accuracy.
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("m,n,k", [(1300, 1310, 2001), (2900, 1025, 1100), (6005, 1400, 3100), (1201, 5000, 6200)])
def test_gemm_split_operands_matches_64_bits(ta, tb, m, n, k):
    from paper_2503_23144_amd import lrcc
    g = torch.Generator(device="cuda:0").manual_seed(m + n + k)
    rand = lambda *s: torch.randn(*s, dtype=torch.complex64, device="cuda:0", generator=g)  # noqa: E731
    A, B, C0 = rand(*((k, m) if ta else (m, k))), rand(*((n, k) if tb else (k, n))), rand(m, n)
    rows = (10.0 ** -(torch.arange(m, device="cuda:0") % 7)).to(torch.complex64)
    A = A * (rows[None, :] if ta else rows[:, None])
    C0 = C0 * rows[:, None]
    al, be = 0.6 - 0.2j, -0.3 + 0.7j
    C = C0.clone()
    lrcc.gemm(A, B, C, transa=bool(ta), transb=bool(tb), alpha=al, beta=be, noalloc=True)
    D = torch.complex128
    ref = al * ((A.T if ta else A).to(D) @ (B.T if tb else B).to(D)) + be * C0.to(D)
    err = (C.to(D) - ref).abs().amax(1) / rows.real.double()
    scale = np.sqrt(k) * 5.0 * 5.0 + 5.0
    assert float(err.max()) <= 20 * 2e-7 * scale * np.sqrt(k)
    # no further from 64 bits than the FP32 matrix cores
    lrcc.gemm_set_tile(0)
    try:
        C2 = C0.clone()
        lrcc.gemm(A, B, C2, transa=bool(ta), transb=bool(tb), alpha=al, beta=be, noalloc=True)
    finally:
        lrcc.gemm_set_tile(-1)
    rel = [float(((x.to(D) - ref).abs() ** 2).sum(1).div((ref.abs() ** 2).sum(1)).sqrt().max()) for x in (C, C2)]
    assert rel[0] <= 1.1 * rel[1], rel


def test_gemm_split_operands_extreme_inputs():
    """Values near the ends of the FP32 range, zeros and infinities."""
    from paper_2503_23144_amd import lrcc
    m = n = 1536
    k = 1536
    z = lambda *s: torch.zeros(*s, dtype=torch.complex64, device="cuda:0")  # noqa: E731
    A, B, C = z(m, k), z(k, n), z(m, n)
    A[0, 0], B[0, 0] = 3.4e38, 0.5         # rounds up to infinity in BF16
    A[1, 1], B[1, 1] = 1.17549435e-38, 1e30  # smallest normal number
    A[2, 2], B[2, 2] = float("inf"), 2.0
    A[3, 3], B[3, 3] = float("nan"), 1.0
    lrcc.gemm(A, B, C, noalloc=True)
    torch.cuda.synchronize()
    c = C.cpu().numpy()
    assert abs(c[0, 0].real - 1.7e38) <= 1e-6 * 1.7e38 and np.isfinite(c[0]).all()
    assert abs(c[1, 1].real - 1.17549435e-8) <= 1e-6 * 1.2e-8
    assert not np.isfinite(c[2, 2]) and not np.isfinite(c[3, 3])
    assert not c[4:].any()


@pytest.mark.parametrize("o,v", [(3, 10), (5, 21), (8, 44)])
def test_small_workflow_repeats_with_graphs(o, v):
    """Small systems read permuted operands in place and share one executor
    between batches of one and three: the truncation workflow and products on
    a side stream give the same results every time, as without graphs."""
    from paper_2503_23144_amd import lrcc
    from paper_2503_23144_amd.synth import make_inputs
    inp = make_inputs(o, v, 2 * v, seed=5)
    om = [0.05]

    def workflow(graphs):
        st = torch.cuda.Stream()
        c = lrcc.Context(stream=st.cuda_stream, graphs=graphs)
        out = []
        for _ in range(4):
            c.load_df(o, v, inp.B)
            c.load_fock(inp.fock)
            c.load_dipoles(inp.mu)
            for _ in range(3):
                e0, a0 = c.mp2_response(om)
            _, occ = c.fnspp_truncate(om, keep=v // 2)
            e1, a1 = c.mp2_response(om)
            out.append(np.concatenate([[e0, e1], occ, a0.ravel(), a1.ravel()]))
        c.close()
        return out

    ref, got = workflow(False), workflow(True)
    for x in got:
        assert np.abs(x - ref[0]).max() <= 1e-12 * np.abs(ref[0]).max()


@pytest.mark.parametrize("o,v,nb", [(9, 53, 20), (17, 37, 18)])
def test_permuted_operands_packed_in_place(o, v, nb):
    """Ring products (K = o v) and the o^2 products (K = o^2 >= 256) of batches
    large enough to pack their operands, read through index maps with odd
    extents.  FP32 against FP64 of the same context: 2^-24 per rounding, sums
    of at most v^2 terms in chains, against the largest element."""
    from paper_2503_23144_amd import lrcc
    from paper_2503_23144_amd.synth import make_inputs
    print(f"packed in place o={o} v={v} nb={nb}", flush=True)
    inp = make_inputs(o, v, o + v, seed=o * v)
    c = lrcc.Context(precision="mixed", tol=1e-9)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    c.load_dipoles(inp.mu)
    rng = np.random.default_rng(o + v)
    t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
    X = rng.standard_normal((nb, c.n)) + 1j * rng.standard_normal((nb, c.n))
    c.sigma("residual", t)
    c.set_amplitudes(lrcc.AMP_T, t)
    for side in ("right", "left"):
        ref = c.sigma(side, X, precision="fp64")
        got = c.sigma(side, X, precision="mixed")
        for r in range(nb):
            assert np.abs(got[r] - ref[r]).max() <= 1e-5 * np.abs(ref[r]).max(), (side, r)
    c.close()


@pytest.mark.parametrize("o,v,nb,precision,tol", [(9, 53, 20, "mixed", 1e-5), (6, 40, 1, "fp64", 1e-12)])
def test_tile_pinned_between_runs(o, v, nb, precision, tol):
    """Pinning a tile after a program's eager run sends its products to other
    kernels, with other scratch: that run is eager again, not a capture.  Both
    sum the same terms in another order (2^-24 or 2^-53 per rounding)."""
    from paper_2503_23144_amd import lrcc
    from paper_2503_23144_amd.synth import make_inputs
    print(f"pinned tile o={o} v={v} nb={nb} {precision}", flush=True)
    inp = make_inputs(o, v, o + v, seed=o * v)
    c = lrcc.Context(precision=precision, tol=1e-9)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    c.load_dipoles(inp.mu)
    rng = np.random.default_rng(o + v)
    t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
    X = rng.standard_normal((nb, c.n)) + 1j * rng.standard_normal((nb, c.n))
    c.sigma("residual", t)
    c.set_amplitudes(lrcc.AMP_T, t)
    try:
        for side in ("left", "right"):
            ref = c.sigma(side, X, precision=precision)
            for tile in (0, 0, 0, -1, -1, -1, 3, -1):
                lrcc.gemm_set_tile(tile)
                got = c.sigma(side, X, precision=precision)
                assert np.abs(got - ref).max() <= tol * np.abs(ref).max(), (side, tile)
    finally:
        lrcc.gemm_set_tile(-1)
    c.close()
