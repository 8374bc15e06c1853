"""The per-wavefront curl kernel (one wavefront per component, LDS exchange of the three
spectra): symmetric and semi-unbounded directions c and b (imaginary factors), tiles of
one, two and four groups of lines with ragged ends, and the planner's choice of it for
FP64 plans of many lines.  Tolerances are those of every parity test (FP64 1e-12, FP32
1e-5 relative L-infinity against the FP64 oracle)."""
import numpy as np
import pytest

import oracle as O
import paper_2211_07777_amd as F
from gpu_common import TOL32, TOL64, rel_linf

pytestmark = pytest.mark.gpu
U, P, E, D = 3, 2, 0, 1


def _faces(sym):
    """Faces per component: axis a of `sym` has normal component faces sym[a], the two
    others the opposite symmetry; the other axes unbounded."""
    swap = {E: D, D: E, U: U}
    return [[[f if q == a else swap[f] for f in sym[a]] if a in sym else [U, U] for a in range(3)] for q in range(3)]


@pytest.mark.parametrize("prec,tol", [(F.F64, TOL64), (F.F32, TOL32)])
@pytest.mark.parametrize("sym", [{0: [E, E]}, {0: [D, E]}, {0: [U, E]}, {0: [E, E], 1: [D, U]}, {1: [E, D], 0: [D, D]}])
@pytest.mark.parametrize("layout", [O.CELL, O.NODE])
def test_symmetric_directions(sym, layout, prec, tol):
    import torch
    n, h = [7, 9, 32], [0.11, 0.09, 1 / 32]
    bcv = _faces(sym)
    f = np.random.default_rng(31 + layout).standard_normal((3,) + O.user_shape(n, layout))
    ref = O.solve_vector(f, n, h, bcv, layout, 0, F.BIOT_SAVART_FD2)
    plan = F.Plan(n, h, bcv, layout, F.CHAT2, prec, F.BIOT_SAVART_FD2)
    t = plan.tiling()
    x = torch.from_numpy(f).to("cuda", plan.dtype).contiguous()
    ran = 0
    for values, mode in ((16, 3), (8, 4)):
        for groups in (1, 2, 4):
            b, q = list(t["lines_per_tile"]), list(t["persistent"])
            b[2], q[2] = groups * 64 * values // 64, mode
            try:
                plan.set_tiling(b, q)
            except F.FluxmiError:
                continue
            u = plan.solve(x)
            torch.cuda.synchronize()
            err = rel_linf(u.double().cpu().numpy(), ref)
            assert err < tol, (sym, layout, mode, groups, err)
            ran += 1
    assert ran >= 3
    plan.close()


@pytest.mark.parametrize("n,wave", [([32, 64, 32], True), ([30, 64, 32], False)])
def test_fp64_default(n, wave):
    """FP64 curl passes of at least 4096 lines (33 x 128 here) run per wavefront without
    tuning, shorter ones (31 x 128) in the LDS-tile kernel."""
    import torch
    h = [1 / 32] * 3
    plan = F.Plan(n, h, [[U, U]] * 3, F.CELL, F.CHAT2, F.F64, F.BIOT_SAVART, 3)
    assert (plan.tiling()["persistent"][2] == 4) == wave
    f = np.random.default_rng(3).standard_normal((3,) + O.user_shape(n, O.CELL))
    u = plan.solve(torch.from_numpy(f).cuda())
    torch.cuda.synchronize()
    assert rel_linf(u.cpu().numpy(), O.solve(f, n, h, [[U, U]] * 3, O.CELL, 0, 1)) < TOL64
    plan.close()
