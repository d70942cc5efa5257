"""The spectral diagnostics by one component at a time, as they run where there is no memory for three,
against the batch of three, on even, odd and thin grids and on every route that fills their fields."""

import pytest
import torch

from parity_helpers import Case, gpu_solver

pytestmark = pytest.mark.gpu
CASES = [Case(16, 12, 10, seed=3), Case(15, 13, 11, seed=4, forced=True), Case(130, 3, 4, seed=5, kmax=1),
         Case(3, 5, 129, seed=6, kmax=1), Case(12, 14, 9, jmode="stencil", seed=7),
         Case(13, 10, 9, seed=8, collision="bgk", fluid_lattice="d3q19"),
         Case(12, 10, 8, seed=9, magnetic_lattice="d3q15")]


@pytest.mark.parametrize("layout", ["aa", "ab"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c.nx}x{c.ny}x{c.nz}-{c.jmode}-{c.fluid_lattice}-{c.magnetic_lattice}")
def test_one_component_matches_three(case, layout, monkeypatch):
    out = {}
    for batch in ("", "1"):
        monkeypatch.setenv("FLAME_SPECTRAL_BATCH", batch)
        s = gpu_solver(case, "f64", layout)
        s.step(3)
        n = max(case.shape) // 2 + 2
        out[batch] = [s.spectrum("u", n), s.spectrum("B", n), s.dissipation_spectrum("u", n),
                      s.dissipation_spectrum("B", n), s.energy_transfer(n, hall=True)]
        for first, again in zip(out[batch], [s.spectrum("u", n), s.spectrum("B", n), s.dissipation_spectrum("u", n),
                                             s.dissipation_spectrum("B", n), s.energy_transfer(n, hall=True)]):
            assert torch.equal(first, again)
        s.close()
    # the same sums in another order: some hundred roundings of the largest shell; the transfer's terms
    # cancel within a shell, so there of the energies times the largest wavenumber
    for three, one in zip(out[""][:4], out["1"][:4]):
        assert float((three - one).abs().max()) <= 1e-13 * float(three.abs().max())
    scale = float(out[""][0].sum() + out[""][1].sum()) * torch.pi
    assert float((out[""][4] - out["1"][4]).abs().max()) <= 1e-13 * scale


def test_one_component_matches_the_oracle(monkeypatch):
    from oracle import diagnostics, scheme
    from parity_helpers import oracle_run
    monkeypatch.setenv("FLAME_SPECTRAL_BATCH", "1")
    case = Case(15, 12, 14, seed=11)
    p, st = oracle_run(case, 2)
    s = gpu_solver(case, "f64", "aa")
    s.step(2)
    _, U, B, J, _ = scheme.fields(st, p)
    for name, v in (("u", U), ("B", B)):
        want = torch.as_tensor(diagnostics.spectrum(v, 9))
        assert float((s.spectrum(name, 9) - want).abs().max()) < 1e-10 * float(want.abs().max())
    got = s.energy_transfer(9)
    want = torch.stack([torch.as_tensor(t) for t in diagnostics.energy_transfer(U, B, J, 9)[:3]])
    scale = float(U.norm() ** 2 + B.norm() ** 2) / U[0].numel() * float(B.abs().max() + U.abs().max())
    assert float((got - want).abs().max()) < 1e-11 * scale
    s.close()
