"""Passes that the planner runs with twiddle tables in LDS (launch modes 1, persistent, and
0) or per wavefront (4) because they are slower with one tile per workgroup and tables from
global memory (mode 2), on both sides of each line; two of the grids against the FP64 oracle
with the tolerances of every parity test."""
import numpy as np
import pytest

import oracle as O
import paper_2211_07777_amd as F
from gpu_common import TOL32, TOL64, rel_linf

pytestmark = pytest.mark.gpu
U, P, E, D = [3, 3], [2, 2], [0, 0], [0, 1]
POIS, CURL = F.POISSON, F.BIOT_SAVART


@pytest.mark.parametrize("n,bc,prec,kind,ncomp,modes", [
    ([96, 96, 96], [U, U, U], F.F32, CURL, 3, {3: 1, 4: 0, 5: 1}),       # lines of 192 points
    ([48, 48, 48], [U, U, U], F.F32, CURL, 3, {3: 2, 4: 0, 5: 1}),       # 96 points, 343 tiles
    ([96, 96, 96], [U, U, U], F.F64, CURL, 3, {3: 1}),
    ([48, 48, 48], [U, U, U], F.F64, CURL, 3, {3: 2}),                   # 96 points
    ([48, 48, 384], [P, U, P], F.F64, POIS, 1, {2: 0, 4: 0}),            # 384 points
    ([384, 96, 96], [P, P, P], F.F32, POIS, 1, {5: 0}),
    ([128, 128, 64], [U, U, U], F.F32, POIS, 3, {4: 1}),                 # 256 points, 1548 tiles
    ([128, 128, 64], [U, U, U], F.F32, POIS, 1, {4: 2}),                 # 516 tiles
    ([192, 192, 192], [D, E, P], F.F64, POIS, 1, {1: 1}),                # 384-point extensions
    ([96, 96, 192], [D, E, P], F.F64, POIS, 1, {1: 2}),
    ([256, 256, 128], [P, P, P], F.F32, POIS, 1, {1: 2, 5: 2}),          # contiguous packed lines
    ([256, 256, 128], [U, P, D], F.F32, POIS, 1, {2: 4, 4: 4}),          # strided ones
    ([512, 128, 128], [P, P, P], F.F32, POIS, 1, {1: 4, 5: 4}),
    ([512, 256, 256], [P, P, P], F.F32, POIS, 1, {1: 1, 5: 4}),          # beyond the cache
    ([128, 128, 64], [D, E, P], F.F64, POIS, 3, {3: 1}),                 # fused packed lines
    ([256, 200, 32], [D, E, P], F.F64, POIS, 1, {3: 2}),                 # 32 points
    ([256, 200, 32], [D, E, P], F.F32, POIS, 1, {3: 2}),
    ([256, 200, 48], [P, P, P], F.F32, POIS, 1, {3: 2}),                 # 48 points
    ([256, 200, 48], [P, P, P], F.F32, CURL, 3, {3: 2}),
    ([128, 128, 64], [D, [1, 1], E], F.F32, POIS, 3, {3: 1}),            # fused real-to-real
    ([256, 200, 32], [D, [1, 1], E], F.F32, POIS, 1, {3: 2}),            # 64 points
])
def test_default_modes(n, bc, prec, kind, ncomp, modes):
    layout = F.NODE if bc == [U, P, D] else F.CELL
    plan = F.Plan(n, [1 / 64] * 3, bc, layout, F.CHAT2, prec, kind, ncomp)
    got = plan.tiling()["persistent"]
    assert {k: got[k - 1] for k in modes} == modes, got
    plan.close()


@pytest.mark.parametrize("n,bc,prec,tol,kind", [
    ([96, 96, 96], [U, U, U], F.F32, TOL32, CURL), ([96, 96, 96], [U, U, U], F.F64, TOL64, CURL),
    ([48, 48, 384], [P, U, P], F.F64, TOL64, POIS), ([384, 96, 96], [P, P, P], F.F32, TOL32, POIS),
])
def test_parity(n, bc, prec, tol, kind):
    import torch
    h, nc = [1 / 64] * 3, 3 if kind == CURL else 1
    f = np.random.default_rng(sum(n)).standard_normal(((nc,) if nc > 1 else ()) + O.user_shape(n, O.CELL))
    plan = F.Plan(n, h, bc, F.CELL, F.CHAT2, prec, kind, nc)
    u = plan.solve(torch.from_numpy(f).to("cuda", plan.dtype).contiguous())
    torch.cuda.synchronize()
    assert rel_linf(u.double().cpu().numpy(), O.solve(f, n, h, bc, O.CELL, 0, kind)) < tol
    plan.close()
