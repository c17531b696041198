"""What a call returns does not depend on what its workspace held: every byte of it
set (any float read from it unwritten is NaN) gives the results of a zeroed one."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1506_02079_amd as gdf
import synth

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _fuse(stack, alpha, tol, bc, precision, fill):
    """fuse_stack with a workspace of bytes `fill`: status, f, reports."""
    S, H, W = stack.shape
    o = gdf.make_opts(precision, out_dtype=gdf.DTYPE_F64)
    L = gdf.lib()
    n = L.gdf_fuse_workspace_size(S, H, W, ctypes.byref(o))
    work = torch.full((n,), fill, dtype=torch.uint8, device=DEV)
    f = torch.zeros((S, H, W), dtype=torch.float64, device=DEV)
    rep = (gdf.SliceReport * S)()
    torch.cuda.synchronize()
    st = L.fuse_stack(stack.data_ptr(), S, H, W, W, H * W, alpha, gdf.BC[bc], tol, 1.0, 3.0, f.data_ptr(), None,
                      ctypes.byref(o), work.data_ptr(), n, rep, None)
    torch.cuda.synchronize()
    return st, f, [(r.vcycles, r.status, r.rel_residual, r.rel_residual_init) for r in rep]


# 8 x 9 x 4 = 288 and 8 x 9 x 5 = 360 row blocks of 64 x 256 (the row-marching output and
# refinement passes start at 256), rows that end 1, 2 and 3 pixels into a lane's
# quad, a last block of one pixel, and whole quads; one small stack
@pytest.mark.parametrize("precision", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("bc,shape", [("neumann", (8, 520, 1021)), ("neumann", (8, 520, 1022)),
                                      ("neumann", (8, 520, 1023)), ("neumann", (8, 520, 1025)),
                                      ("neumann", (8, 520, 1020)), ("periodic", (8, 520, 1021)),
                                      ("neumann", (5, 97, 83)), ("periodic", (5, 97, 83))])
def test_fuse_stack_with_dirty_workspace(bc, shape, precision):
    stack = torch.from_numpy(synth.make_stack(*shape, seed=sum(shape), ramp=True)).to(DEV)
    tol = 1e-9 if precision == "mixed" else 1e-6
    print("dirty workspace", bc, shape, precision, flush=True)
    s0, f0, r0 = _fuse(stack, 0.01, tol, bc, precision, 0)
    s1, f1, r1 = _fuse(stack, 0.01, tol, bc, precision, 255)
    print(r0[0], r1[0], flush=True)
    assert s0 == gdf.GDF_OK and s1 == gdf.GDF_OK
    assert all(np.isfinite(r[2:]).all() and r[2] <= tol for r in r1)
    assert torch.equal(f0, f1) and r0 == r1


@pytest.mark.parametrize("precision", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("sizes", [[(700, 1021), (1500, 1023), (1100, 1026), (700, 2050)], [(1, 1), (33, 70), (129, 5)]])
def test_solve_and_backward_with_dirty_workspace(sizes, precision):
    rng = np.random.default_rng(3)
    dt = torch.float64 if precision == "fp64" else torch.float32
    go = [torch.from_numpy(rng.integers(0, 256, size=s).astype(np.float64)).to(DEV, dt) for s in sizes]
    gs = [o + 9.0 * torch.randn(o.shape, generator=torch.Generator(DEV).manual_seed(4), device=DEV, dtype=dt) for o in go]
    n = len(sizes)
    L = gdf.lib()
    px = [h * w for h, w in sizes]
    got, lam = torch.cat([v.flatten() for v in go]), torch.cat([v.flatten() for v in gs])
    d = (gdf.SliceDesc * n)()
    for i, (h, w) in enumerate(sizes):
        d[i].H, d[i].W, d[i].alpha = h, w, 0.01
        d[i].off_gs = d[i].off_go = d[i].off_f = sum(px[:i])
        d[i].pitch_gs = d[i].pitch_go = d[i].pitch_f = w
    code = gdf.DTYPE_F64 if precision == "fp64" else gdf.DTYPE_F32
    tol = 1e-9 if precision == "mixed" else 1e-6
    out = []
    for fill in (0, 255):
        print("dirty workspace", sizes, precision, fill, flush=True)
        o = gdf.make_opts(precision, out_dtype=gdf.DTYPE_F64)
        ws = L.gdf_solve_workspace_size(n, d, ctypes.byref(o))
        work = torch.full((ws,), fill, dtype=torch.uint8, device=DEV)
        f = torch.zeros(sum(px), dtype=torch.float64, device=DEV)
        rep = (gdf.SliceReport * n)()
        torch.cuda.synchronize()
        st = L.solve_slices(n, d, code, lam.data_ptr(), code, got.data_ptr(), 0, tol, f.data_ptr(), ctypes.byref(o),
                            work.data_ptr(), ws, rep, None)
        # the adjoint of a loss whose gradient is g_s - g_o
        ob = gdf.make_opts("fp64" if precision == "fp64" else "fp32")
        wb = L.gdf_backward_workspace_size(n, d, ctypes.byref(ob))
        work = torch.full((wb,), fill, dtype=torch.uint8, device=DEV)
        grad, fd = lam - got, f.to(dt)
        ggs, ggo = torch.zeros_like(grad), torch.zeros_like(grad)
        ga, repb = (ctypes.c_double * n)(), (gdf.SliceReport * n)()
        torch.cuda.synchronize()
        sb = L.solve_slices_backward(n, d, code, grad.data_ptr(), fd.data_ptr(), lam.data_ptr(), 0, 1e-6, ggs.data_ptr(),
                                     ggo.data_ptr(), ga, None, ctypes.byref(ob), work.data_ptr(), wb, repb, None)
        torch.cuda.synchronize()
        out.append((st, sb, [(r.vcycles, r.rel_residual) for r in rep], [(r.vcycles, r.rel_residual) for r in repb],
                    list(ga), f, ggs, ggo))
    a, b = out
    assert a[0] == a[1] == gdf.GDF_OK
    assert a[:5] == b[:5]
    assert all(torch.equal(x, y) for x, y in zip(a[5:], b[5:]))
