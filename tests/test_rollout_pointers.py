"""What the differentiable rollout hands to the library by pointer, on the CPU with the library stubbed:
dense float64 arrays whatever the strides and type of the caller's tensors, and gradients that come back in
the caller's type."""

import ctypes
import types

import numpy as np
import pytest
import torch

from paper_2212_11024_amd import adjoint

SHAPE = (3, 4, 5)          # nz, ny, nx


class FakeSolver:
    def __init__(self, nx, ny, nz, *args, **kw):
        self.ctx, self.device, self.n = 1, torch.device("cpu"), nx * ny * nz
        self.stream = types.SimpleNamespace(synchronize=lambda: None)

    def step(self, n):
        pass

    def fields(self):
        z = torch.zeros((3,) + SHAPE, dtype=torch.float64)
        return None, z, z, None, None


@pytest.fixture
def handed(monkeypatch):
    seen = {}

    def at(ptr, count):
        return np.ctypeslib.as_array((ctypes.c_double * count).from_address(ptr))

    def adjoint_init(ctx, lam, u, b, gu, gb, out_u, out_b, out_gu, out_gb):
        n = SHAPE[0] * SHAPE[1] * SHAPE[2]
        for name, p, k in (("u", u, 3), ("b", b, 3), ("gu", gu, 9), ("gb", gb, 9)):
            seen[name] = at(p, k * n).copy()
        for p, k in ((out_u, 3), (out_b, 3), (out_gu, 9), (out_gb, 9)):
            at(p, k * n)[:] = np.arange(k * n)

    monkeypatch.setattr(adjoint, "Solver", FakeSolver)
    monkeypatch.setattr(adjoint.L, "flame_trace_bytes", lambda c: 8)
    for name in ("flame_trace_export", "flame_adjoint_fields", "flame_trace_step", "flame_adjoint_trace_step"):
        monkeypatch.setattr(adjoint.L, name, lambda *a: None)
    monkeypatch.setattr(adjoint.L, "flame_adjoint_init", adjoint_init)
    return seen


def _permuted(t):
    return t.movedim(0, -1).contiguous().movedim(-1, 0)


def _expanded(t):
    return t[:, :1].expand_as(t)


@pytest.mark.parametrize("form", [_permuted, _expanded, lambda t: t.float()])
def test_the_library_reads_dense_float64(handed, form):
    g = torch.Generator().manual_seed(2)
    rand = lambda *lead: form(torch.randn(*lead, *SHAPE, dtype=torch.float64, generator=g))  # noqa: E731
    args = [rand(3), rand(3), rand(3, 3), rand(3, 3)]
    leaves = [a.detach().requires_grad_() for a in args]
    cfg = adjoint.RolloutConfig(SHAPE[2], SHAPE[1], SHAPE[0], 0.02, 0.02, nsteps=2)
    u, B = adjoint.FlameRollout.apply(*leaves, cfg)
    (u.sum() + B.sum()).backward()
    for name, a in zip(("u", "b", "gu", "gb"), args):
        assert np.array_equal(handed[name], a.double().contiguous().numpy().reshape(-1)), name
    for leaf in leaves:
        assert leaf.grad.dtype == leaf.dtype
        assert torch.equal(leaf.grad, torch.arange(leaf.numel(), dtype=torch.float64).view(leaf.shape).to(leaf.dtype))


def test_spectral_gradient_is_dense_whatever_the_transform_returns(monkeypatch):
    v = torch.randn(3, *SHAPE, dtype=torch.float64, generator=torch.Generator().manual_seed(3))
    want = adjoint.spectral_gradient(v)
    real = torch.fft.irfftn
    monkeypatch.setattr(torch.fft, "irfftn", lambda *a, **k: _permuted(real(*a, **k)))
    got = adjoint.spectral_gradient(v)
    assert want.is_contiguous() and got.is_contiguous() and torch.equal(got, want)
