"""Slices at the FP32 floor are re-solved in as few solves as their order and the
workspace allow."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1506_02079_amd as gdf

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("large_at", ["last", "first"])
def test_one_large_slice_does_not_split_the_rest(large_at):
    """64 small slices and a large one whose re-solve takes the whole workspace: two
    groups, so three right-hand sides are formed in all (the FP32 solve's included)."""
    sizes = [(40, 40)] * 64 + [(600, 600)]
    if large_at == "first":
        sizes.reverse()
    rng = np.random.default_rng(8)
    go = [torch.from_numpy(rng.integers(0, 256, size=s).astype(np.float32)).to(DEV) for s in sizes]
    gs = [o + torch.from_numpy(rng.normal(0, 20, size=s).astype(np.float32)).to(DEV) for o, s in zip(go, sizes)]
    L = gdf.lib()
    # the workspace is the large slice's re-solve and nothing more
    d = (gdf.SliceDesc * len(sizes))()
    for i, (H, W) in enumerate(sizes):
        d[i].H, d[i].W, d[i].alpha = H, W, 0.01
        d[i].pitch_gs = d[i].pitch_go = d[i].pitch_f = W
    big = (gdf.SliceDesc * 1)(d[0] if large_at == "first" else d[len(sizes) - 1])
    fp32, mixed = gdf.make_opts("fp32"), gdf.make_opts("mixed")
    assert L.gdf_solve_workspace_size(len(sizes), d, ctypes.byref(fp32)) == \
        L.gdf_solve_workspace_size(1, big, ctypes.byref(mixed))
    print("groups, large slice", large_at, flush=True)
    L.gdf_profile_reset()
    L.gdf_profile_enable(1)
    try:
        f, rep = gdf.solve_slices(gs, go, 0.01, tol=1e-12)   # (beyond FP32: every slice is re-solved)
    finally:
        L.gdf_profile_enable(0)
    n = L.gdf_profile_read(b"prep", None, None)
    L.gdf_profile_reset()
    print("right-hand sides", n, flush=True)
    assert all(r["status"] == gdf.GDF_OK and r["rel_residual"] <= 1e-12 for r in rep)
    assert n == 3
