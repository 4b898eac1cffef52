"""GPU: the resident kernel that runs the one-sweep iteration of small grids on
chip, against the oracle and the sweeps it stands in for.

* Fixed counts to the parity bar of fixed-count runs (1e-11 against the
  oracle's iterates) over boxes of every height, grids that end inside a box in
  each direction, non-uniform phi and both upper boundaries.
* Solves that span several launches, and that stop by tolerance, count and
  breakdown, as the sweeps' do.
* The way out when a launch cannot come together (forced by a wait of 0 us):
  the solve is done in sweeps and gives the sweeps' result, alone and in the
  server.
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import GRIDS, check_solution, dev, gpu_solve, iters_close, label, make_faces

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# one box; boxes that end inside the grid in r, theta, phi; phi of one cell past a box
SHAPES = [GRIDS[0], GRIDS[2], GRIDS[4], GRIDS[5], (17, 17, 65, "stretched", "ratio3", "uniform")]


@pytest.mark.parametrize("m", ["1", "2", "4", "8", "16"])
@pytest.mark.parametrize("case", SHAPES, ids=label)
def test_fixed_counts_match_oracle(case, m, monkeypatch):
    monkeypatch.setenv("POT3D_ONCHIP_M", m)
    print(f"[on chip] {label(case)} M={m}", flush=True)
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    for closed in (False, True):
        ref = {K: oracle.solve(rf, tf, pf, br, 0.0, K, closed_wall=closed) for K in (1, 2, 9)}
        upper = P.UPPER_CLOSED_WALL if closed else P.UPPER_SOURCE_SURFACE
        with P.Solver(rf, tf, pf, upper_bc=upper) as s:
            for K, o in ref.items():
                phi, st, it, _ = gpu_solve(s, br, 0.0, K)
                assert st == P.ENOCONV and it == K
                check_solution(phi, o["phi"], tol=1e-11)


@pytest.mark.parametrize("precision", [P.FP64, P.FP32_REFINED], ids=["fp64", "fp32_refined"])
@pytest.mark.parametrize("case", [GRIDS[4], GRIDS[6]], ids=label)
def test_solves_like_the_sweeps(case, precision, monkeypatch):
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    got = {}
    for chip in ("1", "0"):
        monkeypatch.setenv("POT3D_ONCHIP", chip)
        with P.Solver(rf, tf, pf, precision=precision) as s:
            got[chip] = [gpu_solve(s, br, 1e-10, 100_000), gpu_solve(s, br, 1e-10, 7)]
            if precision == P.FP64:
                got[chip].append(gpu_solve(s, br, 0.0, 5000))   # more than one launch
            bad = br.copy()
            bad[2, 3] = np.inf
            got[chip].append(gpu_solve(s, bad, 1e-10, 100))
    a, b = got["1"], got["0"]
    assert [g[1] for g in a] == [g[1] for g in b]
    # FP32 rounding sets how many inner iterations a refined solve adds: no more than the sweeps' 5 % over
    assert iters_close(a[0][2], b[0][2]) if precision == P.FP64 else a[0][2] <= 1.05 * b[0][2]
    assert [g[2] for g in a[1:]] == [g[2] for g in b[1:]]
    check_solution(a[0][0], b[0][0], tol=1e-8 if precision == P.FP64 else 1e-7)
    check_solution(a[1][0], b[1][0], tol=1e-11 if precision == P.FP64 else 1e-5)
    if precision == P.FP64:
        check_solution(a[2][0], b[2][0], tol=1e-10)
        assert a[2][3] <= 2.0 * b[2][3]   # the residual it drifts to


@pytest.mark.parametrize("precision", [P.FP64, P.FP32_REFINED], ids=["fp64", "fp32_refined"])
def test_gives_up_and_sweeps(precision, monkeypatch):
    rf, tf, pf = make_faces(*GRIDS[6])
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    with P.Solver(rf, tf, pf, precision=precision) as s:
        want = gpu_solve(s, br, 1e-10, 100_000)
    monkeypatch.setenv("POT3D_ONCHIP", "1")
    monkeypatch.setenv("POT3D_ONCHIP_WAIT_US", "0")
    with P.Solver(rf, tf, pf, precision=precision) as s:
        first, second = gpu_solve(s, br, 1e-10, 100_000), gpu_solve(s, br, 1e-10, 100_000)
    with P.Server(precision=precision, max_slots=2) as sv:
        ids = [sv.submit(rf, tf, pf, br, 1e-10, 100_000) for _ in range(2)]
        for _ in range(10_000):
            if sv.step()[2] == len(ids):
                break
        served = [sv.take(i) for i in ids]
    for phi, st, it in [first[:3], second[:3]] + [(p, i["status"], i["iters"]) for p, i in served]:
        assert st == P.OK and it == want[2] and np.array_equal(phi, want[0])
