"""The planner's launch modes against the FP64 oracle on both sides of every line that it
draws (sizes, types, precisions), and the launch modes that bring a length of their own (6: a
plain pass in the runtime-length kernel although its length has a kernel; 7, 8: real-to-real
lines of types II and III of half their extension's length): set, solved, taken back.  Tolerances are those of every parity test (FP64 1e-12, FP32 1e-5 relative
L-infinity)."""
import numpy as np
import pytest

import oracle as O
import paper_2211_07777_amd as F
from gpu_common import TOL32, TOL64, check_conventions, gpu_solve, oracle_solve, rel_linf

pytestmark = pytest.mark.gpu
U, P, E, D = 3, 2, 0, 1
PRECS = pytest.mark.parametrize("prec,tol", [(F.F64, TOL64), (F.F32, TOL32)])


def solve_error(plan, f, ref, bc, layout):
    u = gpu_solve(plan, f)
    check_conventions(u, bc, layout)
    return rel_linf(u, ref)


# few lines; lines that fill 256 workgroups; 2^19 and 2^20 points; 256-point packed lines
@PRECS
@pytest.mark.parametrize("n,bc", [([32, 32, 32], [[E, E], [D, D], [E, D]]),
                                  ([48, 32, 64], [[E, U], [D, E], [P, P]]),
                                  ([128, 96, 32], [[E, D], [U, E], [D, D]]),
                                  ([96, 96, 128], [[D, U], [E, E], [E, E]]),
                                  ([128, 64, 128], [[U, U], [U, U], [E, E]]),
                                  ([128, 128, 96], [[U, U], [P, P], [U, U]])])
def test_defaults(n, bc, prec, tol):
    h = [0.09, 0.1, 0.11]
    for layout in (F.CELL, F.NODE):
        f = np.random.default_rng(sum(n) + layout).standard_normal(O.user_shape(n, layout))
        plan = F.Plan(n, h, bc, layout, F.CHAT2, prec)
        err = solve_error(plan, f, oracle_solve(f, n, h, bc, layout), bc, layout)
        t = plan.tiling()
        plan.close()
        assert err < tol, (n, bc, layout, t, err)


# lengths with a compile-time kernel (32 ... 256 points); types I to IV, extensions, both DFTs
@PRECS
@pytest.mark.parametrize("n,bc", [([16, 32, 24], [[E, E], [D, D], [P, P]]),
                                  ([48, 16, 32], [[E, D], [D, E], [U, U]]),
                                  ([64, 24, 16], [[E, U], [U, D], [E, E]]),
                                  ([32, 64, 32], [[P, P], [E, E], [U, U]]),
                                  ([128, 32, 16], [[D, D], [U, U], [P, P]])])
def test_mode_6(n, bc, prec, tol):
    h = [0.09, 0.1, 0.11]
    for layout in (F.CELL, F.NODE):
        f = np.random.default_rng(sum(n) + layout).standard_normal(O.user_shape(n, layout))
        ref = oracle_solve(f, n, h, bc, layout)
        plan = F.Plan(n, h, bc, layout, F.CHAT2, prec)
        t = plan.tiling()
        before = gpu_solve(plan, f)
        taken = 0
        for lines in (1, 2, 5, 8):
            for k in (0, 1, 3, 4):
                b, m = list(t["lines_per_tile"]), list(t["persistent"])
                b[k], m[k] = lines, 6
                try:
                    got = plan.set_tiling(b, m)
                except F.FluxmiError:  # a length without a compile-time kernel is mode 2
                    continue
                assert got["persistent"][k] == 6 and got["lines_per_tile"][k] == lines
                taken += 1
                err = solve_error(plan, f, ref, bc, layout)
                assert err < tol, (n, bc, layout, k, lines, err)
        assert taken
        assert plan.set_tiling(t["lines_per_tile"], t["persistent"]) == t
        assert np.array_equal(gpu_solve(plan, f), before)
        plan.close()


# one set of faces per component: tangential faces of the even-odd axis, all its transforms
@PRECS
@pytest.mark.parametrize("tang,layout", [((E, E), F.CELL), ((D, D), F.NODE), ((E, D), F.CELL), ((D, E), F.NODE),
                                         ((E, U), F.CELL), ((U, D), F.NODE), ((D, E), F.CELL), ((E, D), F.NODE)])
def test_mode_6_components(tang, layout, prec, tol):
    n, h = [32, 15, 12], [0.04, 0.07, 0.08]
    swap = {E: D, D: E, U: U}
    bc = [[[swap[b] for b in tang] if q == 0 else list(tang), [U, U], [U, U]] for q in range(3)]
    f = np.random.default_rng(3).standard_normal((3,) + O.user_shape(n, layout))
    ref = O.solve_vector(f, n, h, bc, layout, 0, F.BIOT_SAVART)
    plan = F.Plan(n, h, bc, layout, F.CHAT2, prec, F.BIOT_SAVART)
    t = plan.tiling()
    for lines in (1, 4, 5):
        for k in (0, 4):
            b, m = list(t["lines_per_tile"]), list(t["persistent"])
            b[k], m[k] = lines, 6
            assert plan.set_tiling(b, m)["persistent"][k] == 6
            err = rel_linf(gpu_solve(plan, f), ref)
            assert err < tol, (k, lines, err)
    plan.close()


# types II and III of 32 ... 512 points, odd line counts, open ends; every mode of the lines
@PRECS
@pytest.mark.parametrize("n,bc", [([32, 9, 64], [[E, E], [D, D], [D, D]]),
                                  ([7, 128, 5], [[P, P], [D, D], [U, U]]),
                                  ([256, 5, 6], [[E, E], [U, U], [P, P]]),
                                  ([5, 512, 3], [[U, U], [E, E], [P, P]]),
                                  ([32, 5, 128], [[E, U], [P, P], [U, D]]),
                                  ([64, 3, 10], [[E, D], [P, P], [P, P]]),
                                  ([3, 64, 10], [[P, P], [D, E], [U, U]]),
                                  ([128, 128, 5], [[U, D], [U, E], [P, P]])])
def test_half_lines_per_wavefront(n, bc, prec, tol):
    taken = set()
    for layout in (F.CELL, F.NODE):
        h = [0.09, 0.1, 0.11]
        f = np.random.default_rng(sum(n) + layout).standard_normal(O.user_shape(n, layout))
        ref = oracle_solve(f, n, h, bc, layout)
        plan = F.Plan(n, h, bc, layout, F.CHAT2, prec)
        t = plan.tiling()
        before = gpu_solve(plan, f)
        for mode in (7, 8):
            for k in (0, 1, 3, 4):
                for lines in (4, 8, 16, 32, 64, 128):
                    b, m = list(t["lines_per_tile"]), list(t["persistent"])
                    b[k], m[k] = lines, mode
                    try:
                        got = plan.set_tiling(b, m)
                    except F.FluxmiError:
                        continue
                    assert got["persistent"][k] == mode and got["lines_per_tile"][k] == lines
                    taken.add((layout, mode, k))
                    err = solve_error(plan, f, ref, bc, layout)
                    assert err < tol, (n, bc, layout, k, mode, lines, err)
        assert plan.set_tiling(t["lines_per_tile"], t["persistent"]) == t
        assert np.array_equal(gpu_solve(plan, f), before)
        plan.close()
    assert {mode for _, mode, _ in taken} == ({7} if 512 in n else {7, 8}), taken


@PRECS
@pytest.mark.parametrize("tang,layout", [((E, E), F.CELL), ((D, D), F.CELL), ((E, D), F.NODE), ((U, D), F.CELL)])
def test_half_lines_components(tang, layout, prec, tol):
    n, h = [64, 15, 12], [0.04, 0.07, 0.08]
    swap = {E: D, D: E, U: U}
    bc = [[[swap[b] for b in tang] if q == 0 else list(tang), [U, U], [U, U]] for q in range(3)]
    f = np.random.default_rng(4).standard_normal((3,) + O.user_shape(n, layout))
    ref = O.solve_vector(f, n, h, bc, layout, 0, F.BIOT_SAVART)
    plan = F.Plan(n, h, bc, layout, F.CHAT2, prec, F.BIOT_SAVART)
    t = plan.tiling()
    taken = 0
    for mode in (7, 8):
        for k in (0, 4):
            for lines in (8, 16, 32, 64, 128):
                b, m = list(t["lines_per_tile"]), list(t["persistent"])
                b[k], m[k] = lines, mode
                try:
                    plan.set_tiling(b, m)
                except F.FluxmiError:
                    continue
                taken += 1
                err = rel_linf(gpu_solve(plan, f), ref)
                assert err < tol, (k, mode, lines, err)
    plan.close()
    assert taken >= 4, taken


@PRECS
def test_components_on_a_persistent_grid(prec, tol):
    """The three components of a pass in one launch, each on more tiles than a third of the
    resident workgroups."""
    n, h = [32, 72, 72], [0.05, 0.04, 0.03]
    bc = [[[D, D] if q == 0 else [E, E], [P, P], [P, P]] for q in range(3)]
    f = np.random.default_rng(6).standard_normal((3,) + O.user_shape(n, F.CELL))
    ref = O.solve_vector(f, n, h, bc, F.CELL, 0, F.BIOT_SAVART)
    plan = F.Plan(n, h, bc, F.CELL, F.CHAT2, prec, F.BIOT_SAVART)
    t = plan.tiling()
    for mode, lines in ((0, 1), (1, 1), (1, 2), (2, 1), (4, None), (6, 1), (8, None)):
        for k in (0, 4):
            b, m = list(t["lines_per_tile"]), list(t["persistent"])
            b[k], m[k] = lines or 64, mode
            assert plan.set_tiling(b, m)["tiles"][k] > (682 if lines else 32)
            err = rel_linf(gpu_solve(plan, f), ref)
            assert err < tol, (mode, lines, k, err)
    plan.close()


def test_large_batches_equal_single_solves_bitwise():
    """A one-launch batch that fills the chip takes larger tiles than the plans of their own."""
    import torch
    from paper_2211_07777_amd import workloads as W
    reqs = W.serving_stream(count=40, qps=1e4, seed=31, edges=(32, 48, 64))
    plans = [F.Plan(r["n"], r["h"], r["bc"], r["layout"], F.CHAT2, F.F64) for r in reqs]
    rhs = [W.request_rhs_device(r, torch.float64) for r in reqs]
    single = [p.solve(x).clone() for p, x in zip(plans, rhs)]
    outs = [torch.empty_like(x) for x in rhs]
    ws = torch.empty(F.batched_workspace_bytes(plans), dtype=torch.uint8, device="cuda")
    batch = F.Batch(plans, rhs, outs, ws)
    batch.run()
    torch.cuda.synchronize()
    batch.close()
    for r, p, a, b in zip(reqs, plans, single, outs):
        assert torch.equal(a, b), (r["n"], r["bc"], r["layout"])
        p.close()
