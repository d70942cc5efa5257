"""Grids at the edges of the kernels' units against the oracle: blocks of consecutive nodes (rows
shorter and longer than a wavefront, a last block with one node), the 64 x 8 and 64 x 4 tiles and plane chunks
of the curl-stencil kernels, and the 64-entry pieces of the spectral binning."""

import pytest
import torch

from parity_helpers import Case, deviation_error, gpu_solver, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["aa", "ab"])
@pytest.mark.parametrize("grid", [(63, 3, 3), (64, 3, 5), (65, 3, 3), (255, 3, 3), (257, 3, 3), (3, 5, 19)])
def test_blocks_of_consecutive_nodes(grid, layout):
    case = Case(*grid, forced=True, seed=5, kmax=1)
    for steps in (1, 4):
        p, st = oracle_run(case, steps)
        s = gpu_solver(case, "f64", layout)
        s.step(steps)
        assert deviation_error(s, p, st) < 1e-12     # the FP64 parity bar
        s.close()


@pytest.mark.parametrize("layout", ["aa", "ab"])
@pytest.mark.parametrize("grid", [(64, 8, 3), (65, 9, 7), (63, 7, 67), (3, 17, 5), (130, 3, 4)])
def test_stencil_tiles(grid, layout):
    from oracle import diagnostics, scheme
    case = Case(*grid, jmode="stencil", forced=True, seed=6, kmax=1)
    for steps in (1, 2):
        p, st = oracle_run(case, steps)
        s = gpu_solver(case, "f64", layout)
        s.step(steps)
        assert deviation_error(s, p, st) < 1e-12
        rho, u, B, J, div = s.fields()
        for got, want in zip((rho, u, B, J), scheme.fields(st, p)):
            assert float((got.cpu() - want).norm() / want.norm()) < 1e-11     # the node fields' bar
        red, want = s.reduce(), torch.as_tensor(diagnostics.reductions(st, p))
        assert float((red[:4] - want[:4]).abs().max() / want[:4].abs().max()) < 1e-11
        assert torch.equal(red, s.reduce())
        s.close()


@pytest.mark.parametrize("grid", [(3, 5, 6), (4, 3, 3), (126, 3, 4), (127, 4, 3), (128, 3, 3), (258, 3, 3)])
def test_spectral_pieces(grid):
    from oracle import diagnostics, scheme
    case = Case(*grid, seed=7, kmax=1)
    p, st = oracle_run(case, 2)
    s = gpu_solver(case, "f64", "aa")
    s.step(2)
    _, U, B, J, _ = scheme.fields(st, p)
    for nshells in (2, max(grid) // 2 + 2):
        for name, v in (("u", U), ("B", B)):
            want = torch.as_tensor(diagnostics.spectrum(v, nshells))
            assert float((s.spectrum(name, nshells) - want).abs().max()) < 1e-10 * float(want.abs().max())
        got = s.energy_transfer(nshells, hall=True)
        want = torch.stack([torch.as_tensor(t) for t in diagnostics.energy_transfer(U, B, J, nshells)[:3]])
        # the largest summand: the terms cancel over the shells of such small grids
        scale = float(U.norm() ** 2 + B.norm() ** 2) / U[0].numel() * float(B.abs().max() + U.abs().max())
        assert float((got[:3] - want).abs().max()) < 1e-11 * scale
        # the kept workspaces give the same bits again, also after another diagnostic used them
        s.spectrum("B", nshells)
        assert torch.equal(got, s.energy_transfer(nshells, hall=True))
    s.close()
