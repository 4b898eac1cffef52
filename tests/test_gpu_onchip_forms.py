"""GPU: every form of a small grid's iteration is the one that runs, and holds.

* pot3d_stats says what ran: boxes of the asked height on chip (sweep_rows 0),
  sweeps where they were asked for.
* Boxes of 16 layers, whose FP64 form keeps x in memory: long runs of several
  launches against the sweeps, to the bars of the other heights' test.
* A solve cut into launches of 256 iterations (the server's) is bit for bit the
  one in launches of 2048, in both precisions and for several heights.
* Small grids in the server's batched sweeps and in the sweeps of the solve
  that allocates nothing, which they reach no more by themselves.
"""
import numpy as np
import pytest

import oracle
from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

import test_zz_no_alloc
from test_gpu_parity import GRIDS, check_solution, gpu_solve, label, make_faces
from test_gpu_serving import MIX, alone, requests, run_server

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

PRECISIONS = pytest.mark.parametrize("precision", [P.FP64, P.FP32_REFINED], ids=["fp64", "fp32_refined"])


@PRECISIONS
@pytest.mark.parametrize("m", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("case", [GRIDS[0], GRIDS[4]], ids=label)
def test_stats_say_what_ran(case, m, precision, monkeypatch):
    rf, tf, pf = make_faces(*case)
    nr, nt, np_ = case[:3]
    br = magnetograms.br_bipoles(tf, pf, 20, seed=8)
    monkeypatch.setenv("POT3D_ONCHIP_M", str(m))
    with P.Solver(rf, tf, pf, precision=precision) as s:
        gpu_solve(s, br, 1e-10, 40)
        st = s.stats()
        columns = -(-nt // 8) * -(-np_ // 64)
        assert (st["sweep_rows"], st["chunk_s"], st["blocks_s"]) == (0, m, columns * -(-nr // m))
        if precision == P.FP64:
            assert st["graph_launches"] == 1
        s.set_iteration(P.ITER_TWO_PASS)
        gpu_solve(s, br, 1e-10, 40)
        assert s.stats()["sweep_rows"] == 4 and s.stats()["iteration"] == P.ITER_TWO_PASS
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    with P.Solver(rf, tf, pf, precision=precision) as s:
        gpu_solve(s, br, 1e-10, 40)
        assert s.stats()["sweep_rows"] == 4 and s.stats()["iteration"] == P.ITER_ONE_SWEEP


@pytest.mark.parametrize("case", [GRIDS[4], GRIDS[6]], ids=label)
def test_sixteen_layers_over_several_launches(case, monkeypatch):
    rf, tf, pf = make_faces(*case)
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    got = {}
    for chip in ("16", "0"):
        monkeypatch.setenv("POT3D_ONCHIP_M" if chip == "16" else "POT3D_ONCHIP", chip)
        with P.Solver(rf, tf, pf) as s:
            got[chip] = gpu_solve(s, br, 0.0, 5000)
            st = s.stats()
        if chip == "16":
            assert st["chunk_s"] == 16 and st["graph_launches"] == 3
    a, b = got["16"], got["0"]
    assert a[1] == b[1] == P.ENOCONV and a[2] == b[2] == 5000
    check_solution(a[0], b[0], tol=1e-10)
    assert a[3] <= 2.0 * b[3]   # the residual it drifts to


@PRECISIONS
@pytest.mark.parametrize("m", ["4", "8", "16"])
def test_launches_continue_bit_for_bit(m, precision, monkeypatch):
    monkeypatch.setenv("POT3D_ONCHIP_M", m)
    reqs = requests([GRIDS[6], GRIDS[4]])
    ref = alone(reqs, precision)
    out, _, _ = run_server(reqs, precision, max_slots=2)
    for (case, rf, tf, pf, br, *_), (phi_a, st_a, it_a, rr_a), (phi_s, info) in zip(reqs, ref, out):
        assert it_a > 256 and info["status"] == st_a == P.OK and info["iters"] == it_a, label(case)
        assert np.array_equal(phi_s, phi_a) and info["relres_true"] == rr_a
        want = oracle.solve(rf, tf, pf, br, 1e-10, 100_000)["phi"]
        check_solution(phi_a, want, tol=1e-8)   # the solve bar of the parity tests


@PRECISIONS
def test_server_batches_unequal_small_grids_in_sweeps(precision, monkeypatch):
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    reqs = requests(MIX)
    ref = alone(reqs, precision)
    out, peak, _ = run_server(reqs, precision, max_slots=3)
    assert peak == 3
    for (phi_a, st_a, it_a, rr_a), (phi_s, info) in zip(ref, out):
        assert info["status"] == st_a == P.OK and info["iters"] == it_a
        assert np.array_equal(phi_s, phi_a) and info["relres_true"] == rr_a


def test_no_alloc_solve_in_sweeps(monkeypatch):
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    test_zz_no_alloc.test_two_calls_second_smaller_then_first_again()
    test_zz_no_alloc.test_closed_wall_and_warm_start()
    test_zz_no_alloc.check((64, 128, 256), 6)
