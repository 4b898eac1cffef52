"""GPU: what follows a launch of the on-chip kernel that gave up (forced by a
wait of 0 us on the launch that does).

* The solve that allocates nothing is done in sweeps and gives their result.
* The device then stays with sweeps for a while (POT3D_ONCHIP_RETRY_MS here,
  otherwise 64 of the waits), for that entry point, for contexts made before
  and after it, and for a server: none of them waits again.  The sweeps and
  the on-chip kernel differ in their last bits, which tells them apart.
* After that time, solves run on chip again.
"""
import time

import numpy as np
import pytest

from paper_1709_01126_amd import pot3d as P
from workloads import magnetograms

from test_gpu_parity import GRIDS, gpu_solve, make_faces
from test_zz_no_alloc import noalloc_solve

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HOLD_MS = 4000


def test_device_stays_with_sweeps_for_a_while(monkeypatch):
    rf, tf, pf = make_faces(*GRIDS[6])
    br = magnetograms.br_bipoles(tf, pf, 30, seed=5)
    go = lambda: noalloc_solve(rf, tf, pf, br, 1e-10, 100_000)  # noqa: E731
    chip = go()
    monkeypatch.setenv("POT3D_ONCHIP", "0")
    sweeps = go()
    with P.Solver(rf, tf, pf) as s:
        swept = gpu_solve(s, br, 1e-10, 100_000)
    monkeypatch.delenv("POT3D_ONCHIP")
    assert not np.array_equal(chip[0], sweeps[0])
    with P.Solver(rf, tf, pf) as early:
        monkeypatch.setenv("POT3D_ONCHIP_WAIT_US", "0")
        monkeypatch.setenv("POT3D_ONCHIP_RETRY_MS", str(HOLD_MS))
        given_up = go()
        t0 = time.monotonic()
        monkeypatch.delenv("POT3D_ONCHIP_WAIT_US")
        monkeypatch.delenv("POT3D_ONCHIP_RETRY_MS")
        second = go()
        first_ctx = gpu_solve(early, br, 1e-10, 100_000)
        with P.Solver(rf, tf, pf) as late:
            new_ctx = gpu_solve(late, br, 1e-10, 100_000)
            with P.Server(max_slots=1) as sv:
                rid = sv.submit(rf, tf, pf, br, 1e-10, 100_000)
                while sv.step()[2] == 0:
                    pass
                served, _ = sv.take(rid)
            assert time.monotonic() - t0 < 1e-3 * HOLD_MS, "too slow for the hold time to tell anything"
            time.sleep(1e-3 * HOLD_MS)
            again, again_ctx = go(), gpu_solve(late, br, 1e-10, 100_000)
    for phi, st, it, _ in (given_up, second):
        assert st == P.OK and it == sweeps[2] and np.array_equal(phi, sweeps[0])
    for got in (first_ctx, new_ctx):
        assert got[1] == P.OK and got[2] == swept[2] and np.array_equal(got[0], swept[0])
    assert np.array_equal(served, swept[0])
    assert again[1] == P.OK and np.array_equal(again[0], chip[0])
    assert again_ctx[1] == P.OK and not np.array_equal(again_ctx[0], swept[0])
