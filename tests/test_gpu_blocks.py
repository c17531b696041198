"""The register-block multigrid passes at the sizes where their tiling can go
wrong: coarse (Neumann) or finest (periodic) sides at and around one region
(128 x 64 cells), the owned parts of the first, middle and last tiles, and
sides of one to three cells.  A seam computed wrongly on a coarse level still
converges, only more slowly, so the cycle counts are bounded as well: the
cycle contracts the residual by 0.15 or better, and 1e-10 takes at most
log(1e-10) / log(0.15) = 12.1, so 13, cycles."""
import numpy as np
import pytest
import torch

import oracle
import paper_1506_02079_amd as gdf

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# sides of level 1 around (rows) 64, 56 + 1, 56 + 48 + 1 and (columns) 128, 120 + 1, 120 + 112 + 1
NEUMANN = [(126, 254), (128, 256), (129, 257), (130, 260), (114, 242), (113, 241), (210, 466), (209, 467), (4, 300),
           (300, 4), (3, 7), (1, 250)]
PERIODIC = [(48, 112), (52, 116), (53, 117), (104, 232), (105, 118), (50, 233), (128, 128), (64, 256), (2, 130), (70, 1)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("bc", ["neumann", "periodic"])
def test_block_tiles_match_oracle(bc, precision):
    sizes = NEUMANN if bc == "neumann" else PERIODIC
    rng = np.random.default_rng(17)
    alpha = 0.004
    go = [rng.integers(0, 256, size=s).astype(np.float64) for s in sizes]
    gs = [(o + rng.normal(0, 20, size=o.shape)).astype(np.float32).astype(np.float64) for o in go]
    tol = 1e-10 if precision == "fp64" else 1e-6
    dt = torch.float64 if precision == "fp64" else torch.float32
    print("blocks", bc, precision, flush=True)
    f, rep = gdf.solve_slices([torch.from_numpy(s).to(DEV, dt) for s in gs], [torch.from_numpy(o).to(DEV, dt) for o in go],
                              alpha, bc=bc, tol=tol, precision=precision, out_dtype=gdf.DTYPE_F64)
    for i, size in enumerate(sizes):
        fi = f[i].cpu().numpy()
        rel = oracle.relres(fi, gs[i], go[i], alpha, bc)
        fr = oracle.solve(gs[i], go[i], alpha, bc, tol=1e-13)
        err = np.linalg.norm(fi - fr)
        # ||f - f*|| <= ||r|| / alpha (the smallest eigenvalue of A); a tenth more for the reference's own residual
        bound = 1.1 * tol * np.linalg.norm(oracle.rhs(gs[i], go[i], alpha, bc)) / alpha
        print(size, "rel %.2e err %.2e bound %.2e cycles %d" % (rel, err, bound, rep[i]["vcycles"]), flush=True)
        assert rep[i]["status"] == gdf.GDF_OK and rel <= 1.01 * tol
        assert err <= bound
        assert precision != "fp64" or rep[i]["vcycles"] <= 13
