"""Rounding of the BGK fluid collision with a force, in FP64 and FP32, over the whole range of the
viscosity: the force must not pass through a term that grows like the viscosity."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from oracle import collision, equilibrium
from oracle.lattice import C, omega_fluid

HERE = os.path.dirname(os.path.abspath(__file__))
D = ctypes.POINTER(ctypes.c_double)


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("bgk") / "bgk.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-host-only", "-x", "hip",
                    os.path.join(HERE, "hostcheck", "bgk_force.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(out)
    lib.bgk_collide.argtypes = [ctypes.c_int] + [D] * 4 + [ctypes.c_double, D]
    return lib


@pytest.mark.parametrize("single", [0, 1])
@pytest.mark.parametrize("nu", [1e-4, 0.02, 1.0 / 6.0, 0.2, 5.0, 1e3, 1e6, 1e9, 1e60])
def test_error_does_not_grow_with_the_viscosity(lib, nu, single):
    rng = np.random.default_rng(3)
    b0 = np.float32([0.01, -0.02, 0.05]).astype(np.float64)
    omega = float(np.float32(omega_fluid(nu))) if single else omega_fluid(nu)
    one = torch.ones(1, dtype=torch.float64)
    rest = equilibrium.f_mhd_eq(one, torch.zeros(3, 1, dtype=torch.float64), torch.tensor(b0).view(3, 1))[:, 0]
    for _ in range(20):
        f = np.float32(rng.normal(0, 1e-2, 27)).astype(np.float64)
        b = np.float32(rng.normal(0, 0.05, 3)).astype(np.float64)
        F = np.float32(rng.normal(0, 1e-3, 3)).astype(np.float64)
        out = np.empty(27)
        lib.bgk_collide(single, *[a.ctypes.data_as(D) for a in (f, b, b0, F)], omega, out.ctypes.data_as(D))
        full = (torch.tensor(f) + rest).view(27, 1)
        rho = full.sum(0)
        U = (torch.einsum("in,ia->an", full, C) + 0.5 * torch.tensor(F).view(3, 1)) / rho
        want = collision.collide_bgk_closed(full, rho, U, torch.tensor(b0 + b).view(3, 1), omega,
                                            F=torch.tensor(F).view(3, 1))[:, 0] - rest
        # about 64 roundings, of values of the size of the deviations (FP32) or of the oracle's full
        # populations, at most 0.3 (FP64)
        bound = 64 * (2.0 ** -24 * 0.05 if single else 2.0 ** -53 * 0.3)
        assert float((torch.tensor(out) - want).abs().max()) < bound, nu
