"""Planning of grids on both sides of 2^31 output elements per tile, the reach of the
per-wavefront kernels' 32-bit offsets: real-to-real and packed DFT passes along z whose
tiles span nearly the whole grid plan with another kernel instead of being refused.
Host-only (no device memory is needed)."""
import pytest

import paper_2211_07777_amd as F
from test_library_host import _create_vector

P, E, D, U = [2, 2], [0, 0], [1, 1], [3, 3]


@pytest.mark.parametrize("prec", [F.F32, F.F64])
@pytest.mark.parametrize("n,z,layout", [
    ([2048, 2048, 256], E, F.CELL), ([2048, 2048, 486], E, F.CELL),  # below 2^31
    ([2048, 2048, 512], E, F.NODE), ([2160, 2048, 512], E, F.CELL), ([2160, 2048, 512], E, F.NODE),
    ([2160, 2048, 512], D, F.CELL), ([4096, 2048, 512], E, F.CELL), ([4096, 4096, 128], E, F.NODE),
    ([4096, 4096, 256], E, F.CELL), ([4000, 3000, 256], D, F.NODE), ([4000, 3000, 256], [0, 3], F.CELL),
    ([4096, 4096, 128], [0, 1], F.CELL), ([4096, 2048, 512], P, F.CELL), ([4096, 4096, 256], P, F.NODE),
])
def test_large_grids_plan(n, z, layout, prec):
    info = F.plan_inspect(n, [1 / 64] * 3, [P, P, z], layout, F.CHAT2, prec)
    assert all(t >= 1 for t in info["tiles"])


@pytest.mark.parametrize("prec", [F.F32, F.F64])
@pytest.mark.parametrize("n,layout", [([4096, 1024, 256], F.NODE), ([4096, 1024, 512], F.NODE), ([4096, 1080, 512], F.CELL)])
def test_large_vector_grids_pass_planning(n, layout, prec):
    normal, other = [P, P, D], [P, P, E]
    # planned; the device is what is missing here (the status of a grid that fits is -6 too)
    assert _create_vector(n, [1 / 64] * 3, [other, other, normal], layout, prec=prec) == -6
