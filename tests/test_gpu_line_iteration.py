"""GPU: the two-kernel iteration with the phi-line preconditioner, where its
wavefronts change hands: row lengths at and around a lane's runs (one cell
short of a run's end, one past it, several cells per lane, the longest row),
polar rows that do not fill the workgroups, more layers than a wavefront
prepares at a time, and chunks of a few layers.

* Fixed counts on both parities of the x pairing against the oracle's
  line-preconditioned iterates.  Bar: 1e-11, the bar of fixed-count runs, or
  where the rows are long K 4 eps / e: the two blocks differ by a few ulps of
  the diagonal d, which moves z = M^-1 r by up to 4 eps / e relative in every
  iteration, e = d / (2 w) - 1 the smallest over the rows.
* The FP32-refined mode meets its tolerance on the same kind of grid.
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import gpu_solve, make_faces

pytestmark = pytest.mark.gpu

CASES = [(3, 5, 63), (70, 6, 65), (4, 3, 700), (3, 5, 1409), (2, 4, 2048)]


def name(case):
    return "x".join(map(str, case))


@pytest.mark.parametrize("ci", ["3", "1000"], ids=["chunks", "one_chunk"])
@pytest.mark.parametrize("case", CASES, ids=name)
def test_fixed_counts(case, ci, monkeypatch):
    monkeypatch.setenv("POT3D_LINE_CI", ci)
    rf, tf, pf = make_faces(*case, "stretched", "ratio3", "uniform")
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    coef = oracle.assemble(rf, tf, pf)
    b = oracle.rhs(rf, tf, pf, br)
    A = oracle.to_sparse(coef).tocsr()
    d = A.diagonal().reshape(case)[:, :, 0].ravel()
    first = np.arange(case[0] * case[1]) * case[2]
    w = -np.asarray(A[first, first + 1]).ravel()
    e = (d / (2.0 * w) - 1.0).min()
    with P.Solver(rf, tf, pf) as s:
        s.set_preconditioner(P.PC_PHI_LINE)
        for K in (1, 2, 3, 6):
            phi, st, it, _ = gpu_solve(s, br, 0.0, K)
            assert st == P.ENOCONV and it == K
            want = oracle.pcg(coef, b, 0.0, K, precond="phi_line")[0]
            err = np.abs(phi - want).max() / np.abs(want).max()
            bar = max(1e-11, K * 4 * np.finfo(float).eps / e)
            print(f"[line iteration] {name(case)} K={K}: {err:.2e} (bar {bar:.1e})", flush=True)
            assert err <= bar


@pytest.mark.parametrize("case", [(70, 6, 65), (4, 5, 700)], ids=name)
def test_refined(case, monkeypatch):
    monkeypatch.setenv("POT3D_LINE_CI", "3")
    rf, tf, pf = make_faces(*case, "stretched", "ratio3", "uniform")
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    coef = oracle.assemble(rf, tf, pf)
    b = oracle.rhs(rf, tf, pf, br)
    with P.Solver(rf, tf, pf, precision=P.FP32_REFINED) as s:
        s.set_preconditioner(P.PC_PHI_LINE)
        phi, st, _, _ = gpu_solve(s, br, 1e-10, 100_000)
    assert st == P.OK and oracle.true_relres(coef, b, phi) <= 1.01e-10
