"""Small ops launched in groups of independent ones against the same ops
launched one by one (per-launch timing keeps them apart)."""
import numpy as np
import pytest

from paper_2503_23144_amd.synth import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mixed", 1e-5)])
@pytest.mark.parametrize("o,v,nb", [(2, 2, 1), (2, 17, 3), (4, 16, 1), (5, 33, 2), (8, 9, 5)])
def test_grouped_runs_match_single_launches(o, v, nb, precision, tol):
    """The order of a run's ops and of each accumulation is the same in both;
    products without a permuted operand run on another kernel, which sums its
    K <= 1024 terms in another order: sqrt(1024) roundings of 2^-53 (2^-24)
    against the largest element, times the depth of the program (< 20)."""
    from paper_2503_23144_amd import lrcc
    print(f"groups o={o} v={v} nb={nb} {precision}", flush=True)
    inp = make_inputs(o, v, o + v, seed=o * v)
    c = lrcc.Context(precision=precision, tol=1e-9)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    c.load_dipoles(inp.mu)
    rng = np.random.default_rng(o + v + nb)
    t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
    X = rng.standard_normal((nb, c.n)) + 1j * rng.standard_normal((nb, c.n))
    calls = [lambda: c.sigma("residual", t), lambda: c.sigma("right", X, precision=precision),
             lambda: c.sigma("left", X, precision=precision)]
    c.set_timing(True)
    c.sigma("residual", t)
    c.set_amplitudes(lrcc.AMP_T, t)
    ref = [f() for f in calls]
    c.set_timing(False)
    for run in range(4):  # eager, captured, replayed
        for f, r in zip(calls, ref):
            assert np.abs(f() - r).max() <= tol * np.abs(r).max(), run
    c.close()


@pytest.mark.parametrize("o,v", [(2, 3), (3, 31), (2, 32), (3, 33), (2, 65)])
def test_summed_packs_match_oracle_at_tile_edges(o, v):
    """The packs that end the right program and the unpacks that start the left
    one share launches over 32 x 32 tiles of the virtual pair.  FP64 sums of at
    most v^2 + o v < 5000 terms, sqrt(5000) * 2^-53 < 1e-14, times the depth of
    the program (< 20), against the largest element."""
    import torch

    from oracle.response import Problem, left_sigma, right_sigma
    from paper_2503_23144_amd import lrcc
    print(f"packs o={o} v={v}", flush=True)
    inp = make_inputs(o, v, o + v, seed=o * v)
    P = Problem.from_arrays(inp.B, inp.fock, inp.mu, inp.o)
    c = lrcc.Context(precision="fp64", tol=1e-11)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    c.load_dipoles(inp.mu)
    rng = np.random.default_rng(o + v)
    t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
    X = rng.standard_normal((2, c.n)) + 1j * rng.standard_normal((2, c.n))
    c.sigma("residual", t)
    c.set_amplitudes(lrcc.AMP_T, t)
    for side, fn in (("right", right_sigma), ("left", left_sigma)):
        got = c.sigma(side, X)
        for r in range(2):
            ref = fn(P, torch.as_tensor(t), torch.as_tensor(X[r])).resolve_conj().numpy()
            assert np.abs(got[r] - ref).max() <= 1e-12 * np.abs(ref).max(), (side, r)
    c.close()


@pytest.mark.parametrize("o,v", [(8, 9), (4, 16), (9, 15)])
def test_deep_products_cut_along_k_match_oracle(o, v):
    """Depths o^2 v and o v^2 of 576 to 2025 on a few tiles: pieces of 256, the
    last one ragged.  The same check and bound."""
    test_summed_packs_match_oracle_at_tile_edges(o, v)
