"""Node-local steps on either side of the sizes where their stores and their reserved LDS change: against the
oracle on sampled nodes, and the state-saving step against the plain one, bitwise."""

import pytest
import torch

from paper_2212_11024_amd import _lib as L
from paper_2212_11024_amd.solver import Solver
from parity_helpers import sampled_step_error

pytestmark = pytest.mark.gpu
B0 = (0.01, -0.02, 0.05)


def _solver(n, storage, layout="aa"):
    g = torch.Generator(device="cuda").manual_seed(4)
    u, b = (0.02 * torch.randn(3, n, n, n, dtype=torch.float64, device="cuda", generator=g) for _ in range(2))
    return Solver(n, n, n, 0.02, 0.03, 2.0, B0, storage, "moment", layout, u, b)


@pytest.mark.parametrize("n,storage,bar", [(118, "f32", 1e-5), (128, "f32", 1e-5), (130, "f32", 1e-5), (100, "f64", 1e-12),
                                           (106, "f64", 1e-12)])
def test_in_place_steps_at_the_sizes_where_the_stores_change(n, storage, bar):
    s = _solver(n, storage)
    centres = [(0, 0, 0), (n - 1, n - 1, n - 1), (n // 2, 0, n - 1), (63, 64, 1), (n - 2, 17, n // 2)]
    for _ in range(3):                       # even, odd, even
        err, worst = sampled_step_error(s, centres, n, 0.02, 0.03, 2.0, B0)
        assert err < bar and worst < 10 * bar
    s.close()


@pytest.mark.parametrize("layout", ["aa", "ab"])
@pytest.mark.parametrize("n,storage", [(48, "f32"), (112, "f32"), (128, "f32"), (136, "f32"), (140, "f16"), (146, "f16"),
                                       (88, "f64"), (104, "f64"), (128, "f64")])
def test_saving_steps_advance_like_plain_ones(n, storage, layout):
    plain, saving = _solver(n, storage, layout), _solver(n, storage, layout)
    A = torch.float64 if storage == "f64" else torch.float32
    state = torch.empty(51, n, n, n, dtype=A, device="cuda")
    for _ in range(3):
        before = torch.cat([t.reshape(-1, n, n, n) for t in plain.get_populations(deviations=True)])
        J = plain.fields()[3]
        plain.step(1)
        L.flame_step_save(saving.ctx, state.data_ptr())
        assert torch.equal(state[:48], before.to(A))
        assert float((state[48:] - J).norm() / J.norm()) < (1e-11 if storage == "f64" else 1e-5)
        for a, b in zip(plain.get_populations(deviations=True), saving.get_populations(deviations=True)):
            assert torch.equal(a, b)
    plain.close()
    saving.close()
