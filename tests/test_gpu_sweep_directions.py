"""GPU: the one-sweep iteration carries the last two search directions in a
ring of three buffers and rebuilds the residual from them.

* Fixed counts that end at every place of the ring (and on both parities of
  the x pairing) against the oracle's iterates, to the parity bar of
  fixed-count runs (1e-11), on grids with one and several radial chunks.
* The residual it drifts to: run far past convergence, ||b - A Phi|| / ||b||
  stays within a factor of 2 of what the two-pass iteration, which stores r,
  reaches on the same data (each form rounds r once more per step than the
  other at no more than the size of the update's own rounding).
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import GRIDS, check_solution, gpu_solve, label, make_faces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ci", ["3", "1000"], ids=["chunks", "one_chunk"])
@pytest.mark.parametrize("case", [GRIDS[3], GRIDS[4], GRIDS[5]], ids=label)
def test_every_place_of_the_ring(case, ci, monkeypatch):
    monkeypatch.setenv("POT3D_SWEEP_CI", ci)
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    coef = oracle.assemble(rf, tf, pf)
    b = oracle.rhs(rf, tf, pf, br)
    with P.Solver(rf, tf, pf, iteration=P.ITER_ONE_SWEEP) as s:
        for K in range(1, 8):
            phi, st, it, _ = gpu_solve(s, br, 0.0, K)
            assert st == P.ENOCONV and it == K
            check_solution(phi, oracle.pcg(coef, b, 0.0, K)[0], tol=1e-11)


@pytest.mark.parametrize("case", [GRIDS[4], GRIDS[6]], ids=label)
def test_limiting_residual_matches_the_stored_one(case, monkeypatch):
    monkeypatch.setenv("POT3D_SWEEP_ROWS", "4")
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    rr = {}
    for form in (P.ITER_ONE_SWEEP, P.ITER_TWO_PASS):
        with P.Solver(rf, tf, pf, iteration=form) as s:
            rr[form] = gpu_solve(s, br, 1e-15, 3000)[3]
    print(f"[limiting residual] {label(case)} {rr}", flush=True)
    assert np.isfinite(rr[P.ITER_ONE_SWEEP]) and rr[P.ITER_ONE_SWEEP] <= 2.0 * rr[P.ITER_TWO_PASS]


@pytest.mark.parametrize("np_", [50, 56, 105, 113])
def test_tile_widths(np_, monkeypatch):
    """Rows of one 56-cell tile (short of it, and exactly), of one and a part,
    and rows that stay on 48-cell tiles: the oracle's iterates to the same bar."""
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    rf, tf, pf = make_faces(20, 29, np_, "stretched", "ratio3", "jittered")
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    coef = oracle.assemble(rf, tf, pf)
    b = oracle.rhs(rf, tf, pf, br)
    with P.Solver(rf, tf, pf, iteration=P.ITER_ONE_SWEEP) as s:
        for K in (1, 2, 5, 8):
            phi, st, it, _ = gpu_solve(s, br, 0.0, K)
            assert st == P.ENOCONV and it == K
            check_solution(phi, oracle.pcg(coef, b, 0.0, K)[0], tol=1e-11)
