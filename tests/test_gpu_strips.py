"""Level 0 of large batches: the fused finest passes as marched strips, and the
row-marching output pass against the quad one.  A given item height sends a batch of
any size through the strips, so small ones reach every variant of an item (interior,
column edge, guarded) here, in both precisions."""
import numpy as np
import pytest
import torch

import oracle
import paper_1506_02079_amd as gdf

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# columns around one strip of 128 less its halo of 2 (sweeps + 2) on either side, rows
# around items of 16 and their halo, odd and very short sides
SIZES = [(300, 412), (97, 203), (128, 128), (129, 105), (60, 104), (61, 97), (257, 3), (3, 257), (2, 700), (700, 2), (47, 1000)]


def _pairs(sizes, dt, seed):
    rng = np.random.default_rng(seed)
    go = [rng.integers(0, 256, size=s).astype(np.float64) for s in sizes]
    gs = [(o + rng.normal(0, 20, size=o.shape)).astype(np.float32).astype(np.float64) for o in go]
    return go, gs, [torch.from_numpy(o).to(DEV, dt) for o in go], [torch.from_numpy(s).to(DEV, dt) for s in gs]


@pytest.mark.parametrize("precision,nu,sweeps,sor", [(p, n, s, False) for p in ("fp64", "fp32")
                                                     for n, s in ((1, 2), (1, 3), (1, 4), (2, 4), (2, 5), (2, 6))]
                         + [("fp32", 2, 4, True), ("fp32", 2, 5, True), ("fp32", 1, 4, True)])
@pytest.mark.parametrize("tile_rows", [16, 80])
def test_strips_match_oracle(tile_rows, precision, nu, sweeps, sor):
    alpha = 0.004
    dt = torch.float64 if precision == "fp64" else torch.float32
    go, gs, to, ts = _pairs(SIZES, dt, 19)
    tol = 1e-10 if precision == "fp64" else 1e-6
    print("strips", tile_rows, precision, nu, sweeps, sor, flush=True)
    f, rep = gdf.solve_slices(ts, to, alpha, tol=tol, precision=precision, out_dtype=gdf.DTYPE_F64, tile_rows=tile_rows,
                              nu=nu, fine_sweeps=sweeps, sor=sor)
    for i, size in enumerate(SIZES):
        fi = f[i].cpu().numpy()
        rel = oracle.relres(fi, gs[i], go[i], alpha)
        fr = oracle.solve(gs[i], go[i], alpha, tol=1e-13)
        err = np.linalg.norm(fi - fr)
        # ||f - f*|| <= ||r|| / alpha (the smallest eigenvalue of A); a tenth more for the reference's own residual
        bound = 1.1 * tol * np.linalg.norm(oracle.rhs(gs[i], go[i], alpha)) / alpha
        print(size, "rel %.2e err %.2e bound %.2e cycles %d" % (rel, err, bound, rep[i]["vcycles"]), flush=True)
        assert rep[i]["status"] == gdf.GDF_OK and rel <= 1.01 * tol
        assert err <= bound
    # the same sweeps as blocks: the same cycles (a slice at the tolerance may differ by one in FP32)
    _, repb = gdf.solve_slices(ts, to, alpha, tol=tol, precision=precision, out_dtype=gdf.DTYPE_F64, nu=nu,
                               fine_sweeps=sweeps, sor=sor)
    diff = [abs(a["vcycles"] - b["vcycles"]) for a, b in zip(rep, repb)]
    assert max(diff) <= (1 if precision == "fp32" else 0) and sum(diff) <= 1


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("go_dtype", [torch.uint8, torch.float32])
def test_row_and_quad_passes_agree(go_dtype, precision):
    """A batch above the 256 row blocks from which the marching passes run, and the same
    batch after a 3 x 3 slice, which sends the whole call through the quad passes."""
    sizes = [(700, 1020 + k) for k in range(5)] + [(1100, 255), (1100, 257), (1500, 4), (900, 5), (63, 513), (640, 2048)]
    assert sum(-(-H // 64) * (-(-W // 256)) for H, W in sizes) >= 256
    dt = torch.float64 if precision == "fp64" else torch.float32
    al = [0.02] + [0.005 + 0.003 * i for i in range(len(sizes))]
    _, _, to, ts = _pairs([(3, 3)] + sizes, dt, 23)
    to = [t.to(go_dtype) for t in to]
    print("row vs quad passes", precision, go_dtype, flush=True)
    kw = dict(tol=1e-6, precision=precision, out_dtype=gdf.DTYPE_F64)
    f1, r1 = gdf.solve_slices(ts[1:], to[1:], al[1:], **kw)
    f2, r2 = gdf.solve_slices(ts, to, al, **kw)
    # The sums of b are added in another order: its mean, which is removed in the
    # working precision, may round differently (FP32: a rounding of values to 255,
    # 1.5e-5 each way), and so may the residual, whose rounding part is 1e-8.
    for i, size in enumerate(sizes):
        a, b = r1[i], r2[i + 1]
        err = float((f1[i] - f2[i + 1]).abs().max())
        print(size, "max difference %.2e residuals %.6e %.6e" % (err, a["rel_residual"], b["rel_residual"]), flush=True)
        assert a["vcycles"] == b["vcycles"] and a["status"] == b["status"] == gdf.GDF_OK
        assert abs(a["rel_residual_init"] - b["rel_residual_init"]) <= 1e-12 * a["rel_residual_init"]
        assert err <= (1e-9 if precision == "fp64" else 3e-5)
        assert abs(a["rel_residual"] - b["rel_residual"]) <= (1e-6 * a["rel_residual"] if precision == "fp64" else 1e-8)
