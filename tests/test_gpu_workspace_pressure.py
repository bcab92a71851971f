"""Contexts in a workspace that just holds a product, or does not."""
import numpy as np
import pytest
import torch

from paper_2503_23144_amd.synth import make_inputs

pytestmark = pytest.mark.gpu

O, V, FEW, MANY = 12, 90, 8, 200


@pytest.fixture(scope="module")
def system():
    inp = make_inputs(O, V, 60, seed=1)
    rng = np.random.default_rng(2)
    n = O * V + (O * (O - 1) // 2) * (V * (V - 1) // 2)
    t = 0.01 * (rng.standard_normal(n) + 1j * rng.standard_normal(n))
    g = torch.Generator(device="cuda:0").manual_seed(3)
    X = torch.randn(MANY, n, dtype=torch.complex128, device="cuda:0", generator=g)
    return inp, t, X


def _context(system, bytes_):
    from paper_2503_23144_amd import lrcc
    inp, t, X = system
    buf = torch.empty(bytes_, dtype=torch.uint8, device="cuda:0")
    c = lrcc.Context(precision="mixed", tol=1e-9, ladder_fp64="direct", rhs_chunk=MANY)
    c.set_workspace(buf)
    c.load_df(inp.o, inp.v, inp.B)
    c.load_fock(inp.fock)
    c.set_amplitudes(lrcc.AMP_T, t)
    return c


def test_calls_after_a_failed_allocation(system):
    """A product that does not fit fails with LRCC_E_NOMEM wherever its memory
    ends, and leaves a context whose next product is right or fails alike."""
    from paper_2503_23144_amd import lrcc
    X = system[2]
    c = _context(system, 24 << 30)
    ref = c.sigma("right", X[:FEW], precision="mixed")
    low = c.workspace_peak()
    c.sigma("right", X, precision="mixed")
    high = c.workspace_peak()
    c.close()
    failed = 0
    for part in np.linspace(0.1, 0.95, 12):
        size = int(low + part * (high - low))
        print(f"workspace of {size} bytes", flush=True)
        c = _context(system, size)
        for _ in range(2):
            for vecs in (X[:FEW], X, X[:FEW]):
                try:
                    got = c.sigma("right", vecs, precision="mixed")
                except lrcc.LrccError as e:
                    assert e.code == lrcc.E_NOMEM
                    failed += 1
                    continue
                d = (got[:FEW] - ref).abs().max()
                assert float(d) <= 1e-5 * float(ref.abs().max())
        c.close()
    assert failed > 0


def test_packed_operands_yield_to_larger_batches(system):
    """Memory that a product took for packed operands is no obstacle to a
    later one: a workspace that holds the large batch on its own, with 6 % to
    spare for the holes that growing buffers leave, holds it after a smaller one,
    too, and again from a recorded graph."""
    from paper_2503_23144_amd import lrcc
    X = system[2]
    c = _context(system, 24 << 30)
    ref = c.sigma("right", X, precision="mixed")
    size = 2 * c.workspace_peak()
    c.close()

    def runs(size, calls):
        c = _context(system, size)
        try:
            for vecs in calls:
                got = c.sigma("right", vecs, precision="mixed")
                assert float((got - ref[:len(vecs)]).abs().max()) <= 1e-5 * float(ref.abs().max())
            return True
        except lrcc.LrccError as e:
            assert e.code == lrcc.E_NOMEM
            return False
        finally:
            c.close()

    tight = []
    while runs(size, [X]):
        tight.append(size)
        size = int(size * 0.97)
    assert tight
    for size in [s for s in tight if s >= 1.06 * tight[-1]][-3:]:
        print(f"workspace of {size} bytes", flush=True)
        assert runs(size, [X[:40], X, X, X, X[:40], X]), size
