"""GPU: operator and preconditioners on input and output arrays that overlap in
part: bit for bit what they return for separate arrays (equal pointers stay
refused).  The arrays are two stretches of one buffer, apart by a cell, a part
of a row, a row, and a layer and a cell, the output before or after the input.
"""
import numpy as np
import pytest

from paper_1709_01126_amd import pot3d as P

from test_gpu_parity import make_faces

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(5, 17, 63), (4, 16, 64)]   # padded rows and rows that need none


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_overlapping_input_and_output(shape):
    nr, nt, np_ = shape
    n = nr * nt * np_
    x = torch.from_numpy(np.random.default_rng(3).standard_normal(n)).to("cuda:0")
    with P.Solver(*make_faces(*shape, "stretched", "ratio3", "uniform")) as s:
        for what in ("apply", "jacobi", "line"):
            if what == "line":
                s.set_preconditioner(P.PC_PHI_LINE)
            call = s.apply if what == "apply" else s.precondition
            want = torch.empty_like(x)
            call(x, want)
            for shift in (1, np_ - 3, np_, nt * np_ + 1):
                for x_first in (True, False):
                    buf = torch.zeros(n + shift, dtype=torch.float64, device="cuda:0")
                    d_x, d_y = (buf[:n], buf[shift:]) if x_first else (buf[shift:], buf[:n])
                    d_x.copy_(x)
                    torch.cuda.synchronize()
                    call(d_x, d_y)
                    assert torch.equal(d_y, want), (what, shift, x_first)
            with pytest.raises(ValueError):
                call(x, x)
