"""A node with an infinite population has no velocity: its node fields, spectra, reductions and field
adjoint are NaN there, as the oracle's sum over all velocities gives (0 times an infinity is NaN), on
every route and layout."""

import pytest
import torch

from paper_2212_11024_amd import _lib as L
from parity_helpers import Case, gpu_solver

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("jmode,layout", [("moment", "aa"), ("moment", "ab"), ("stencil", "aa"), ("stencil", "ab")])
@pytest.mark.parametrize("storage,q,value", [("f64", 0, float("inf")), ("f32", 1, float("-inf")), ("f16", 0, 1e30)])
def test_an_infinite_population_makes_the_node_nan(storage, q, value, jmode, layout):
    s = gpu_solver(Case(6, 5, 7, jmode=jmode, seed=8, kmax=1), storage, layout)
    f, g = s.get_populations(deviations=True)
    f[q, 3, 2, 1] = value                     # beyond the range of FP16, so stored as an infinity there
    s.set_populations(f, g, deviations=True)
    rho, u, B, J, _ = s.fields()
    assert not torch.isfinite(rho[3, 2, 1])
    assert torch.isnan(u[:, 3, 2, 1]).all()
    u[:, 3, 2, 1] = 0
    assert torch.isfinite(u).all() and torch.isfinite(B).all()
    red = s.reduce(allow_nonfinite=True)
    assert red[8] == 1 and torch.isnan(red[0])
    assert torch.isnan(s.spectrum("u", 4)).all()
    assert torch.isfinite(s.spectrum("B", 4)).all()
    one = torch.ones(3 * s.n, dtype=torch.float64, device="cuda")
    lam = torch.empty(48 * s.n, dtype=torch.float64 if storage == "f64" else torch.float32, device="cuda")
    L.flame_adjoint_fields(s.ctx, one.data_ptr(), one.data_ptr(), lam.data_ptr())
    lam = lam.view(48, *s.shape)
    assert torch.isnan(lam[:27, 3, 2, 1]).all()
    assert int((~torch.isfinite(lam)).sum()) == 27
    s.close()
