"""The workspace an autotuned call asks for holds every setting it may try (host
only: the size queries launch nothing)."""
import ctypes
import itertools

import pytest

import paper_1506_02079_amd as gdf


def _candidates(base):
    """Every setting the header names, for the fields left at 0."""
    for nu in [base.nu] if base.nu else [2, 1]:
        for fs, cs, tr, la in itertools.product([base.fine_sweeps] if base.fine_sweeps else [0, 2 * nu, 2 * nu + 1, 2 * nu + 2],
                                                [base.coarse_sweeps] if base.coarse_sweeps else [0, nu, nu + 1],
                                                [base.tile_rows] if base.tile_rows else [0, 32, 64, 128, 256],
                                                [base.launch_mode] if base.launch_mode else [1, 2]):
            c = gdf.SolveOpts.from_buffer_copy(base)
            c.autotune, c.nu, c.fine_sweeps, c.coarse_sweeps, c.tile_rows, c.launch_mode = 0, nu, fs, cs, tr, la
            yield c


@pytest.mark.parametrize("precision", ["fp32", "fp64", "mixed"])
@pytest.mark.parametrize("sizes", [[(96, 80)] * 6, [(1024, 1024)] * 3, [(229, 165)], [(129, 99), (60, 101), (300, 7)],
                                   [(100, 400)], [(1, 1)]])
@pytest.mark.parametrize("fixed", [{}, {"launch_mode": 2}, {"tile_rows": 64}, {"nu": 1}])
def test_autotuned_query_covers_every_candidate(sizes, precision, fixed):
    L = gdf.lib()
    n = len(sizes)
    d = (gdf.SliceDesc * n)()
    for i, (H, W) in enumerate(sizes):
        d[i].H, d[i].W, d[i].alpha = H, W, 0.01
        d[i].pitch_gs = d[i].pitch_go = d[i].pitch_f = W
    o = gdf.make_opts(precision, autotune=True)
    for k, v in fixed.items():
        setattr(o, k, v)
    queries = [lambda q: L.gdf_solve_workspace_size(n, d, ctypes.byref(q)),
               lambda q: L.gdf_backward_workspace_size(n, d, ctypes.byref(q)),
               lambda q: L.gdf_fuse_workspace_size(n, *sizes[0], ctypes.byref(q))]
    for query in queries:
        asked = query(o)
        assert asked >= max(query(c) for c in _candidates(o)) > 0
