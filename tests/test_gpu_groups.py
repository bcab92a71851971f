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
