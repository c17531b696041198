"""Smoothing of stacks whose rows start on any byte: the same values bit for bit as
the aligned loads give, and the oracle's at widths around a tile and its halo."""
import numpy as np
import pytest
import torch

import oracle
import paper_1506_02079_amd as gdf

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("z_range", [None, (2, 4)])
@pytest.mark.parametrize("W", [4, 64, 72, 76, 132])
def test_unaligned_rows_equal_aligned(W, z_range, precision):
    rng = np.random.default_rng(W)
    st = torch.from_numpy(rng.integers(0, 256, size=(6, 53, W), dtype=np.uint8)).to(DEV)
    kw = dict(return_smooth=True, z_range=z_range, precision=precision, allow_noconv=True)
    f0, _, g0 = gdf.fuse_stack(st, 0.01, **kw)
    for off in (1, 2, 3):
        buf = torch.full((6, 53, W + off + 2), 255, dtype=torch.uint8, device=DEV)
        view = buf[:, :, off:off + W]
        view.copy_(st)
        print("unaligned", W, z_range, precision, off, flush=True)
        f1, _, g1 = gdf.fuse_stack(view, 0.01, **kw)
        assert torch.equal(g0, g1) and torch.equal(f0, f1)


@pytest.mark.parametrize("W", [1, 2, 3, 5, 6, 7, 63, 65, 66, 67, 71, 73, 129, 201])
def test_any_width_matches_oracle(W):
    rng = np.random.default_rng(W)
    st = rng.integers(0, 256, size=(4, 31, W), dtype=np.uint8)
    print("width", W, flush=True)
    _, _, g = gdf.fuse_stack(torch.from_numpy(st).to(DEV), 0.01, return_smooth=True, allow_noconv=True)
    # (sums of up to 19 + 7 + 7 positive FP32 terms, values to 255: 33 x 6e-8 x 255)
    assert np.abs(g.cpu().numpy() - oracle.smooth(st)).max() <= 5.1e-4
