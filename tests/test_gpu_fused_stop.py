"""Where solves whose smoothing restricts the right-hand side stop: by one rule at
every screening weight, and no closer to tol than leaves f at the accuracy of FP32."""
import numpy as np
import pytest
import torch

import oracle
import paper_1506_02079_amd as gdf
import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("shape,seed", [((5, 401, 333), 2), ((9, 300, 412), 2), ((6, 200, 260), 1)])
def test_same_cycles_at_neighbouring_weights(shape, seed):
    """alpha differing by 1e-9 of itself changes no residual by more than about that:
    the same cycles, and f equal but for FP32 rounding (values to 255: 1.5e-5 an ulp)."""
    st = torch.from_numpy(synth.make_stack(*shape, seed=seed, ramp=True)).to(DEV)
    print("neighbouring weights", shape, flush=True)
    f0, r0 = gdf.fuse_stack(st, 0.01)
    for a in (0.01 * (1 - 1e-9), 0.01 * (1 + 1e-9)):
        f1, r1 = gdf.fuse_stack(st, a)
        print([r["vcycles"] for r in r0], [r["vcycles"] for r in r1], flush=True)
        assert [r["vcycles"] for r in r0] == [r["vcycles"] for r in r1]
        assert float((f0 - f1).abs().max()) <= 1e-4


@pytest.mark.parametrize("alpha", [0.015, 0.02])
def test_error_at_fp32_accuracy(alpha):
    """A stack whose slices need a fourth cycle for tol: f within 8 units of FP32
    roundoff (2^-24) of the 64-bit solution, relative, in every slice (a slice that
    stops after three, just inside tol, is 20 off)."""
    stack = synth.make_stack(9, 300, 412, seed=1, ramp=True)
    f, rep = gdf.fuse_stack(torch.from_numpy(stack).to(DEV), alpha)
    fr, _ = oracle.fuse_stack(stack, alpha, tol=1e-13)
    e = [np.linalg.norm(a - b) / np.linalg.norm(b) for a, b in zip(f.cpu().numpy().astype(np.float64), fr)]
    print(alpha, [r["vcycles"] for r in rep], ["%.1e" % v for v in e], flush=True)
    assert max(e) <= 8 * 2.0 ** -24


@pytest.mark.parametrize("alpha", [0.003, 0.006, 0.01, 0.02])
def test_no_cycle_more_than_tol_needs(alpha):
    """A slice that took c cycles is not well inside tol after c - 1: the stop in the
    loop is tol but for the rounding of its FP32 residual (a few 2^-24, 0.2 tol)."""
    st = torch.from_numpy(synth.make_stack(24, 384, 448, seed=1001, ramp=True)).to(DEV)
    cycles = [r["vcycles"] for r in gdf.fuse_stack(st, alpha)[1]]
    print(alpha, cycles, flush=True)
    for c in sorted(set(cycles)):
        _, rep = gdf.fuse_stack(st, alpha, max_vcycles=c - 1, allow_noconv=True)
        rel = [r["rel_residual"] for r, k in zip(rep, cycles) if k == c]
        print(c - 1, ["%.2e" % v for v in rel], flush=True)
        assert min(rel) > 0.8e-6
