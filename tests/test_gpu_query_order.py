"""The gather kernels' query order (strips of rows) and head pairs at sizes where they can go wrong: levels
whose last strip has 1 to 7 rows or is the only one, one-pixel-wide levels, odd head counts (no pairs),
levels that end inside a wave. Tolerances are those of the parity tests."""
import pytest

from paper_2505_14022_amd import workloads
from gpu_util import check_parity, require_gpu

CASES = [
    # dtype, N, M, D, levels (grids of at least 1024 workgroups, where strips are used)
    ("f16", 2, 4, 32, ((71, 97), (36, 49), (9, 1), (1, 7))),
    ("f16", 3, 5, 32, ((58, 90), (15, 23))),
    ("f16", 4, 6, 24, ((64, 64), (7, 5))),
    ("f32", 2, 4, 32, ((65, 61), (33, 31), (17, 16))),
    ("f32", 3, 3, 16, ((81, 90), (8, 8), (2, 3))),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}_M{c[2]}_D{c[3]}_{c[4][0][0]}x{c[4][0][1]}")
def test_strips_and_head_pairs(case):
    require_gpu()
    dtype, N, M, D, levels = case
    S = sum(h * w for h, w in levels)
    w = workloads.Workload(f"strips_{dtype}_S{S}", N=N, M=M, D=D, shapes=levels, P=3, Lq=S, dtype=dtype,
                           refs="own_pixel", offset_px=2.0, index=40)
    check_parity(workloads.generate(w), workspace="owner")
