"""The one-launch binning of small problems (a workgroup per batch item, head and level) at the sizes where it can
go wrong: sample counts around the thread count and at the largest that the path takes (and one more), one-pixel
and one-tile levels, many levels, channel counts that are no multiple of its blocks, samples all in one cell or
all off the map. Tolerances are those of the parity tests."""
import numpy as np
import pytest

from paper_2505_14022_amd import msda, workloads
from gpu_util import TOL_GRAD_ATTN, TOL_GRAD_LOC, TOL_GRAD_VALUE, check_parity, require_gpu

CASES = [
    # N, M, D, levels, P, Lq, dtype
    (2, 3, 36, ((5, 9), (3, 2)), 1, 1023, "f32"),
    (1, 2, 64, ((17, 8), (8, 17), (1, 1)), 1, 1024, "f16"),
    (1, 2, 100, ((9, 9),), 1, 1025, "f32"),
    (1, 1, 32, ((40, 33), (8, 8), (1, 3)), 4, 4096, "f32"),     # 16384 samples per level
    (1, 1, 32, ((40, 33), (8, 8), (1, 3)), 5, 3277, "f32"),     # 16385: the many-workgroup passes
    (1, 1, 4, tuple((k + 1, 16 - k) for k in range(16)), 2, 700, "f32"),
    (3, 5, 48, ((31, 23), (16, 12), (8, 6)), 3, 999, "f16"),
    (1, 1, 32, ((120, 200),), 4, 4000, "f32"),                  # 375 tiles, few samples each
    # more than 64 work items for each of 2048 waves, the last ones past the words that a wave holds ahead:
    # 139264 one-pixel tiles with all channels (their second 32 are a remainder of 16), and 8192 tiles in 17 blocks
    (1088, 8, 48, ((1, 1),) * 16, 1, 2, "f32"),
    (64, 8, 516, ((1, 1),) * 16, 1, 2, "f16"),
    # more than 8192 tiles of few records: all channels
    (18, 8, 80, ((9, 9),) * 16, 1, 20, "f16"),
    # the same of rows that are no whole 64-byte pieces: blocks
    (18, 8, 68, ((9, 9),) * 16, 1, 20, "f32"),
    # and of more than 32 records: blocks of channels
    (18, 8, 40, ((9, 9),) * 16, 1, 140, "f32"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"D{c[2]}_L{len(c[3])}_P{c[4]}_Lq{c[5]}_{c[6]}")
def test_small_bins(case):
    require_gpu()
    N, M, D, levels, P, Lq, dtype = case
    check_parity(workloads.random_case(N, M, D, levels, P, Lq, dtype=dtype, seed=D + Lq), workspace="owner")


@pytest.mark.gpu
@pytest.mark.parametrize("where", ["one_cell", "off_map"])
def test_small_bins_degenerate(where):
    require_gpu()
    inp = workloads.random_case(1, 2, 32, ((24, 24), (12, 12)), 4, 1500, seed=9)
    if where == "one_cell":  # every sample of a level in the cell that four tiles share
        inp.loc[..., 0, :, :] = np.float32(8.25 / 24)
        inp.loc[..., 1, :, :] = np.float32(8.25 / 12)
    else:
        inp.loc[...] = np.float32(-0.5)
    check_parity(inp, workspace="owner")


# Sparse problems where "auto" bins slab by slab (their atomics would outlast it), beside the same calls on atomics
# (no workspace).
ROUTES = [
    # N, M, D, levels, P, Lq, dtype, "auto" has a workspace
    (8, 8, 32, ((100, 134), (50, 67), (25, 34), (13, 17)), 4, 300, "f32", True),
    (3, 16, 48, ((61, 83), (31, 41)), 4, 350, "f16", True),
    (8, 8, 32, ((100, 134), (50, 67), (25, 34), (13, 17)), 4, 60, "f16", False),
    (1, 8, 32, ((119, 195), (59, 98), (29, 49)), 2, 1956, "f16", False),  # atomics are as fast, within a fifth
    (2, 3, 36, ((17, 23), (9, 11)), 4, 1500, "f32", True),
]


def host_sizes(case):
    import torch

    N, M, D, levels, P, Lq, _, _ = case
    shapes = torch.tensor(levels)
    area = shapes.prod(1)
    starts = torch.cumsum(area, 0) - area
    return [msda.workspace_size(shapes, starts, N, int(area.sum()), M, D, Lq, len(levels), P, 0, mode)
            for mode in (msda.MSDA_WORKSPACE_PREFERRED, msda.MSDA_WORKSPACE_OWNER)]


@pytest.mark.parametrize("case", ROUTES, ids=lambda c: f"N{c[0]}_M{c[1]}_Lq{c[5]}")
def test_preferred_route(case):
    preferred, owner = host_sizes(case)
    assert owner > 0 and preferred == (owner if case[7] else 0)


@pytest.mark.gpu
@pytest.mark.parametrize("case", ROUTES, ids=lambda c: f"N{c[0]}_M{c[1]}_Lq{c[5]}")
def test_routes_agree(case):
    """Each route against the others: sums of the same fp32 terms in different orders, so within
    the parity bounds."""
    import torch

    require_gpu()
    N, M, D, levels, P, Lq, dtype, _ = case
    inp = workloads.random_case(N, M, D, levels, P, Lq, dtype=dtype, seed=D + Lq)
    t = {k: torch.from_numpy(np.ascontiguousarray(getattr(inp, k))).cuda()
         for k in ("value", "loc", "attn", "grad_out")}
    shapes = torch.tensor(levels)
    area = shapes.prod(1)
    starts = torch.cumsum(area, 0) - area

    def run(workspace):
        return msda.backward(t["value"], shapes, starts, t["loc"], t["attn"], t["grad_out"], workspace=workspace)

    want = run(None)
    for got in (run("auto"), run("owner")):
        for g, w, tol in zip(got, want, (TOL_GRAD_VALUE, TOL_GRAD_LOC, TOL_GRAD_ATTN)):
            assert float((g - w).abs().max()) <= tol * float(w.abs().max())
