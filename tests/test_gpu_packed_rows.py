"""GPU: the entry points that work on the caller's packed rows without copies.

* The operator and both preconditioners at row lengths around a tile's edges
  (63, 64, 65 cells, odd and even) on buffers that start 8 bytes past a
  16-byte boundary: the parity bars of their own tests.
* Nothing is written beyond the caller's arrays, and a solve's state survives
  the calls (its field is the same before and after).
* The host solve copies rows that need no padding (64 cells) and rows that do
  (63) bit for bit as the device solve returns them, with a starting guess.
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import dev, gpu_solve, make_faces

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(5, 17, 63), (3, 16, 64), (4, 15, 65), (2, 33, 128)]


def offset_buffer(n, fill):
    """A packed array of n doubles that starts at an odd multiple of 8 bytes, with guards around it."""
    whole = torch.full((n + 64,), fill, dtype=torch.float64, device="cuda:0")
    assert whole.data_ptr() % 16 == 0
    return whole, whole[33:33 + n]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_operator_and_preconditioners(shape):
    rf, tf, pf = make_faces(*shape, "stretched", "ratio3", "uniform")
    n = int(np.prod(shape))
    coef = oracle.assemble(rf, tf, pf)
    x = np.random.default_rng(5).standard_normal(shape)
    want = {"apply": oracle.matvec(coef, x), "jacobi": x / oracle.to_sparse(coef).diagonal().reshape(shape),
            "line": oracle.line_solve(coef, x)}
    scale = {"apply": (abs(oracle.to_sparse(coef)) @ np.abs(x).ravel()).reshape(shape)}
    br = magnetograms.br_bipoles(tf, pf, 10, seed=2)
    with P.Solver(rf, tf, pf) as s:
        gpu_solve(s, br, 1e-10, 10_000)
        before = [b.clone() for b in s.field()]
        for what in ("apply", "jacobi", "line"):
            if what == "line":
                s.set_preconditioner(P.PC_PHI_LINE)
            _, d_x = offset_buffer(n, 0.0)
            d_x.copy_(torch.from_numpy(x.ravel()))
            whole, d_y = offset_buffer(n, 7.0)
            (s.apply if what == "apply" else s.precondition)(d_x, d_y)
            torch.cuda.synchronize()
            got = d_y.cpu().numpy().reshape(shape)
            # the bars of the operator's and the preconditioner's own parity tests
            bound = 1e-13 * scale.get(what, np.abs(want[what]).max())
            assert np.all(np.abs(got - want[what]) <= bound + 1e-12 * np.abs(want[what]).max() * (what == "line")), what
            assert bool((whole[:33] == 7.0).all()) and bool((whole[33 + n:] == 7.0).all()), what
        after = s.field()
    for a, b in zip(before, after):
        assert torch.equal(a, b)


@pytest.mark.parametrize("np_", [63, 64])
def test_host_copies(np_):
    shape = (6, 9, np_)
    rf, tf, pf = make_faces(*shape, "stretched", "ratio3", "uniform")
    br = magnetograms.br_bipoles(tf, pf, 10, seed=2)
    phi0 = np.random.default_rng(1).standard_normal(shape)
    with P.Solver(rf, tf, pf) as s:
        a = s.solve(br, 0.0, 9, phi0=phi0)
        b = gpu_solve(s, br, 0.0, 9, phi0=phi0)
    assert a[1] == b[1] and a[2] == b[2] == 9 and np.array_equal(a[0], b[0])
