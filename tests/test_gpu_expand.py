"""The tiled expansion of the lean layout's packed block at the edges of its
32 x 32 tiles, against the default layout, which stores every dense block."""
import numpy as np
import pytest

from paper_2503_23144_amd.synth import make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [None, 256])
@pytest.mark.parametrize("o,v", [(2, 2), (3, 31), (2, 32), (3, 33), (33, 34), (5, 65)])
def test_lean_sigma_matches_default_layout(monkeypatch, o, v, chunk):
    """Both layouts sum the same products in FP64, of at most v^2 + o v terms:
    the order differs, sqrt(5000) * 2^-53 < 1e-14 per sum, and the largest
    element is compared."""
    from paper_2503_23144_amd import lrcc
    if chunk is not None:  # one occupied index per chunk: shifted blocks, accumulated and split outputs
        monkeypatch.setenv("LRCC_VIRTUAL_CHUNK_BYTES", str(chunk))
    inp = make_inputs(o, v, o + v, seed=o * v)
    out = {}
    for memory in ("lean", "resident"):
        print(f"expand o={o} v={v} chunk={chunk} {memory}", flush=True)
        c = lrcc.Context(precision="fp64", tol=1e-11, memory=memory)
        c.load_df(inp.o, inp.v, inp.B)
        c.load_fock(inp.fock)
        c.load_dipoles(inp.mu)
        rng = np.random.default_rng(o + v)
        t = 0.05 * (rng.standard_normal(c.n) + 1j * rng.standard_normal(c.n))
        X = rng.standard_normal((2, c.n)) + 1j * rng.standard_normal((2, c.n))
        res = [c.sigma("residual", t)]
        c.set_amplitudes(lrcc.AMP_T, t)
        res += [c.sigma("right", X), c.sigma("left", X)]
        out[memory] = res
        c.close()
    for a, b in zip(out["lean"], out["resident"]):
        assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()
