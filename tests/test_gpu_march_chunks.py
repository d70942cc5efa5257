"""Node fields and reductions of the curl-stencil route over several planes per workgroup: chunks of 2 to 16
planes with a ragged last one, partial tiles in x and y, and more tiles times chunks than the reduction has
blocks, against the oracle's formulas on the run's own populations."""

import pytest
import torch

from oracle import diagnostics, scheme
from parity_helpers import Case, gpu_solver, inputs, oracle_params
from test_node_blocks_host import nb  # noqa: F401

# grid, planes per workgroup and work items on 256 compute units (the reductions have 2048 blocks)
GRIDS = [((3, 64, 130), 4, 528), ((66, 63, 67), 4, 544), ((3, 256, 130), 2, 4160), ((3, 1024, 61), 16, 1024)]


@pytest.mark.parametrize("grid,planes,items", GRIDS)
def test_the_grids_march(grid, planes, items, nb):  # noqa: F811
    nx, ny, nz = grid
    tiles = -(-nx // 64) * -(-ny // 4)
    assert nb.nb_march_planes(tiles, nz, 256 * 4, 32) == planes and tiles * -(-nz // planes) == items


@pytest.mark.gpu
@pytest.mark.parametrize("storage,layout", [("f64", "aa"), ("f32", "ab"), ("f16", "aa")])
@pytest.mark.parametrize("grid", [g[0] for g in GRIDS])
def test_fields_and_reductions_over_chunks(grid, storage, layout):
    nx, ny, nz = grid
    case = Case(*grid, jmode="stencil", forced=True, seed=12, kmax=1)
    fu, fb = inputs(case)[4:]
    ftype = torch.float64 if storage == "f64" else torch.float32
    p = oracle_params(case, fu.to(ftype).double(), fb.to(ftype).double())
    s = gpu_solver(case, storage, layout)
    for _ in range(2):                       # both parities of the in-place layout
        s.step(1)
        st = scheme.State(*(t.cpu() for t in s.get_populations()))
        want, got = scheme.fields(st, p), s.fields()
        for w, g in zip(want[:4], got[:4]):
            assert float((g.cpu() - w).norm() / w.norm()) < 1e-11     # the node fields' bar
        assert float((got[4].cpu() - want[4]).abs().max()) < 1e-13    # a difference of populations of 0.01
        red, ref = s.reduce(), torch.as_tensor(diagnostics.reductions(st, p))
        energy = float(ref[:2].max())
        n = nx * ny * nz
        scale = torch.tensor([energy] * 3 + [float(ref[3])] + [1e-2] * 2 + [float(ref[6]), 1e-2, 0.0] + [n] * 7)
        assert ((red - ref).abs() <= 1e-11 * scale).all(), (red - ref) / scale
        assert torch.equal(red, s.reduce())
    s.close()
