"""FP64 one-launch batches take larger tiles than the plans they hold, also of lengths
without a compile-time kernel: every solve equals the plan's own bitwise, at counts on both
sides of the rule, with odd numbers of lines (two real lines share a transform), all kinds
of lines and the curl."""
import numpy as np
import pytest

import paper_2211_07777_amd as F

pytestmark = pytest.mark.gpu
U, P, E, D = [3, 3], [2, 2], [0, 0], [0, 1]


@pytest.mark.parametrize("count", [1, 2, 5, 24])
@pytest.mark.parametrize("n,bc,kind", [
    ([24, 20, 18], [U, U, U], F.POISSON), ([25, 21, 15], [U, P, U], F.POISSON), ([36, 25, 30], [D, P, U], F.POISSON),
    ([27, 35, 20], [E, D, [1, 3]], F.POISSON), ([20, 45, 21], [E, E, P], F.POISSON), ([9, 90, 7], [P, E, U], F.POISSON),
    ([24, 20, 18], [U, U, U], F.BIOT_SAVART), ([15, 12, 175], [P, U, U], F.BIOT_SAVART)])
def test_batch_equals_singles(n, bc, kind, count):
    import torch
    for layout in (F.CELL, F.NODE):
        plan = F.Plan(n, [0.05] * 3, bc, layout, F.CHAT2, F.F64, kind)
        f = [torch.from_numpy(np.random.default_rng(k).standard_normal(plan.shape)).cuda() for k in range(count)]
        singles = [plan.solve(x) for x in f]
        outs = [torch.empty_like(x) for x in f]
        plans = [plan] * count
        ws = torch.empty(F.batched_workspace_bytes(plans), dtype=torch.uint8, device="cuda")
        F.solve_batched(plans, f, outs, ws)
        torch.cuda.synchronize()
        for s, o in zip(singles, outs):
            assert torch.isfinite(o).all() and torch.equal(s, o), (layout, (s - o).abs().max())
        plan.close()
