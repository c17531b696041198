"""Smoothing of stacks thinner than the cross-slice radius: fewer slices take
kernels of a smaller radius; every thickness around the switch must match the
oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1506_02079_amd as gdf
import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("S", [1, 2, 3, 9, 10, 11])
@pytest.mark.parametrize("precision,robust", [("fp32", False), ("fp64", False), ("fp32", True)])
def test_thin_stack_smoothing(S, precision, robust):
    stack = synth.make_stack(S, 45, 77, seed=300 + S)
    _, _, gsm = gdf.fuse_stack(torch.from_numpy(stack).to(DEV), 0.01, precision=precision, robust=robust,
                               return_smooth=True)
    ref = oracle.smooth_robust(stack) if robust else oracle.smooth(stack)
    d = np.abs(gsm.cpu().numpy() - ref)
    tol = 1e-9 if precision == "fp64" else 2e-4
    # (robust: a value within rounding of the two-deviation threshold may go either way)
    assert (d > tol).mean() <= (2e-3 if robust else 0.0), d.max()
