"""FP64 three-component lines of 1024 points (a 512-cell unbounded axis) per wavefront, with
no, one or two symmetric axes (the default from 4096 lines on): against the FP64 oracle
(1e-12 relative L-infinity, as every FP64 parity test), and against the runtime-length
kernel on the same plan.  With a semi-unbounded axis beside the long unbounded one the
Green's tables of library and oracle differ by up to 2e-12, whichever kernel runs (the
runtime-length kernel's result is as far off), so that set is held to the second check."""
import numpy as np
import pytest

import oracle as O
import paper_2211_07777_amd as F
from gpu_common import TOL64, rel_linf
from test_gpu_wave_curl import D, E, U, _faces

pytestmark = pytest.mark.gpu
# two FP64 transforms of 1024 points and their inverses: a few units in the last place per
# radix stage (at most 5 each way), with a margin of six
KERNELS = 64 * 2.0 ** -52


@pytest.mark.parametrize("sym", [{}, {0: [E, E]}, {0: [E, E], 1: [D, D]}, {0: [D, E], 1: [U, E]}])
@pytest.mark.parametrize("layout", [O.CELL, O.NODE])
def test_1024_point_lines(sym, layout):
    import torch
    n, h = [6, 5, 512], [0.11, 0.09, 1 / 512]
    bcv = _faces(sym)
    f = np.random.default_rng(5 + layout).standard_normal((3,) + O.user_shape(n, layout))
    plan = F.Plan(n, h, bcv if sym else [[U, U]] * 3, layout, F.CHAT2, F.F64, F.BIOT_SAVART, 3)
    t = plan.tiling()
    b, q = list(t["lines_per_tile"]), list(t["persistent"])
    x = torch.from_numpy(f).cuda()
    b[2], q[2] = 1, 3
    plan.set_tiling(b, q)
    u = plan.solve(x).cpu().numpy()
    if not any(U in faces for faces in sym.values()):
        ref = O.solve_vector(f, n, h, bcv, layout, 0, F.BIOT_SAVART) if sym else O.solve(f, n, h, [[U, U]] * 3, layout, 0, 1)
        assert rel_linf(u, ref) < TOL64
    b[2], q[2] = 1, 2
    plan.set_tiling(b, q)
    assert rel_linf(u, plan.solve(x).cpu().numpy()) < KERNELS
    plan.close()


@pytest.mark.parametrize("sym", [{}, {0: [E, E]}, {0: [E, E], 1: [D, D]}])
def test_default(sym):
    n = [64, 64, 512]  # 65 x 65 lines and more
    plan = F.Plan(n, [1 / 64] * 3, _faces(sym) if sym else [[U, U]] * 3, F.CELL, F.CHAT2, F.F64, F.BIOT_SAVART, 3)
    assert plan.tiling()["persistent"][2] == 3
    plan.close()
