"""Three-component lines in the runtime-length kernel: in place (tiles up to 8 points per
thread of 512 threads) at lengths around its workgroup sizes, with tiles of the planner and
of one line, with two buffers beyond 4096 points, and in FP64 batches (whose kernel always
has two buffers), against the FP64 oracle with the tolerances of every parity test."""
import numpy as np
import pytest

import oracle as O
import paper_2211_07777_amd as F
from gpu_common import TOL32, TOL64, rel_linf

pytestmark = pytest.mark.gpu
BC = [[3, 3]] * 3


# unbounded cells; FFT lengths 2 n: 18, 90, 250, 640 (256 threads), 686 (512), 1080, 1350
@pytest.mark.parametrize("prec,tol", [(F.F64, TOL64), (F.F32, TOL32)])
@pytest.mark.parametrize("cells", [9, 45, 125, 320, 343, 540, 675])
def test_in_place(cells, prec, tol):
    import torch
    n, h = [6, 5, cells], [0.05] * 3
    f = np.random.default_rng(cells).standard_normal((3,) + O.user_shape(n, O.CELL))
    ref = O.solve(f, n, h, BC, O.CELL, 0, F.BIOT_SAVART)
    plan = F.Plan(n, h, BC, O.CELL, F.CHAT2, prec, F.BIOT_SAVART, 3)
    t = plan.tiling()
    x = torch.from_numpy(f).to("cuda", plan.dtype).contiguous()
    ran = 0
    for lines in sorted({t["lines_per_tile"][2], 1, 2, 3, 5, 10}):
        b, q = list(t["lines_per_tile"]), list(t["persistent"])
        b[2], q[2] = lines, 2
        try:
            plan.set_tiling(b, q)
        except F.FluxmiError:
            continue
        u = plan.solve(x)
        torch.cuda.synchronize()
        assert rel_linf(u.double().cpu().numpy(), ref) < tol, lines
        ran += 1
    assert ran >= 1
    if prec == F.F64:
        outs = [torch.empty_like(x) for _ in range(2)]
        plan.set_tiling(t["lines_per_tile"], t["persistent"])
        ws = torch.empty(F.batched_workspace_bytes([plan, plan]), dtype=torch.uint8, device="cuda")
        F.solve_batched([plan, plan], [x, x], outs, ws)
        torch.cuda.synchronize()
        for o in outs:
            assert rel_linf(o.cpu().numpy(), ref) < tol
    plan.close()
