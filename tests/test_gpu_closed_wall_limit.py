"""GPU: the on-chip kernel with the closed upper wall, long past convergence.

A's null space holds the constants there.  Rounding puts a little of them into
the residual, which the iteration can't reduce; once the rest of the residual
is smaller, directions and steps grow without bound unless that part is taken
out.  So: fixed counts of several times the iterations to 1e-13, over several
launches, keep the true residual where the oracle's solve to 1e-13 leaves it
(within the 2x of the bar for open walls) and Phi at the oracle's (the solve
bar), for every box height, and tolerances below the rounding of b - A Phi
(1e-16) are still reached by the recursive residual.  In refined mode, whose
outer residual is computed in FP64 and corrected, it stays below 1e-12.
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import GRIDS, check_solution, gpu_solve, label, make_faces
from test_zz_no_alloc import noalloc_solve

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

CASES = pytest.mark.parametrize("case", [GRIDS[4], GRIDS[5], GRIDS[6]], ids=label)


@pytest.mark.parametrize("m", ["2", "4", "8", "16"])
@CASES
def test_long_past_convergence(case, m, monkeypatch):
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    ref = oracle.solve(rf, tf, pf, br, 1e-13, 100_000, closed_wall=True)
    want, limit = ref["phi"], 2.0 * ref["true_relres"]
    monkeypatch.setenv("POT3D_ONCHIP_M", m)
    with P.Solver(rf, tf, pf, upper_bc=P.UPPER_CLOSED_WALL) as s:
        _, st, it, _ = gpu_solve(s, br, 1e-13, 100_000)
        assert st == P.OK and s.stats()["chunk_s"] == int(m) and s.stats()["sweep_rows"] == 0
        for factor in (1.3, 1.6, 2, 3, 5):
            phi, st, _, rr = gpu_solve(s, br, 0.0, int(factor * it))
            assert st == P.ENOCONV and rr <= limit, (factor, rr)
            check_solution(phi, want)
        phi, st, _, rr = gpu_solve(s, br, 1e-16, 100_000)
        assert st == P.OK and rr <= limit
        check_solution(phi, want)


@CASES
def test_refined_long_past_convergence(case):
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    want = oracle.solve(rf, tf, pf, br, 1e-12, 100_000, closed_wall=True)["phi"]
    with P.Solver(rf, tf, pf, upper_bc=P.UPPER_CLOSED_WALL, precision=P.FP32_REFINED) as s:
        for maxit in (1500, 4000):
            phi, _, _, rr = gpu_solve(s, br, 0.0, maxit)
            assert s.stats()["sweep_rows"] == 0 and rr <= 1e-12, (maxit, rr)
            check_solution(phi, want)


@CASES
def test_no_alloc_below_rounding(case):
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    phi, st, _, rr = noalloc_solve(rf, tf, pf, br, 1e-16, 100_000, upper=P.UPPER_CLOSED_WALL)
    ref = oracle.solve(rf, tf, pf, br, 1e-13, 100_000, closed_wall=True)
    assert st == P.OK and rr <= 2.0 * ref["true_relres"]
    check_solution(phi, ref["phi"])
