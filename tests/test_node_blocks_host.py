"""Index arithmetic of the kernels whose blocks own consecutive nodes (division by a row and by a plane,
the 27 periodic neighbours), and the plane count of the marching kernels, on the host."""

import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def nb(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("nb") / "nb.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-host-only", "-x", "hip",
                    os.path.join(HERE, "hostcheck", "node_blocks.hip"), "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(out)
    lib.nb_divide.restype = ctypes.c_uint32
    lib.nb_divide.argtypes = [ctypes.c_uint32, ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    lib.nb_march_planes.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int64, ctypes.c_int]
    lib.nb_neighbours.argtypes = [ctypes.c_int] * 3 + [ctypes.c_uint32, ctypes.POINTER(ctypes.c_uint32)]
    return lib


def test_division_is_exact(nb):
    rng = np.random.default_rng(0)
    rest = ctypes.c_uint32()
    top = 2 ** 32 - 1
    divisors = [1, 2, 3, 5, 64, 65, 257, 65535, 65536, 65537, 2 ** 31 - 1, 2 ** 31, top - 1, top]
    divisors += [int(d) for d in rng.integers(1, top, 200)]
    for d in divisors:
        near = [k * d + e for k in (0, 1, 2, top // d) for e in (-1, 0, 1)]
        for t in [t for t in near if 0 <= t <= top] + [0, top] + [int(v) for v in rng.integers(0, top, 20)]:
            assert (nb.nb_divide(t, d, ctypes.byref(rest)), rest.value) == divmod(t, d), (t, d)


@pytest.mark.parametrize("grid", [(1, 1, 1), (1, 1, 7), (1, 6, 1), (9, 1, 1), (2, 2, 2), (3, 5, 4), (64, 2, 3),
                                  (65, 3, 2), (257, 2, 2), (2048, 1024, 1024)])
def test_neighbours(nb, grid):
    nx, ny, nz = grid
    n = nx * ny * nz
    cells = range(n) if n <= 2000 else [0, 1, nx - 1, nx, nx * ny - 1, nx * ny, n // 2 - 1, n - nx, n - 1]
    out = (ctypes.c_uint32 * 27)()
    for cell in cells:
        nb.nb_neighbours(nx, ny, nz, cell, out)
        z, r = divmod(cell, nx * ny)
        y, x = divmod(r, nx)
        want = [(((z + dz) % nz) * ny + (y + dy) % ny) * nx + (x + dx) % nx
                for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
        assert list(out) == want, cell


def test_march_planes_fill_the_chip(nb):
    for tiles, nz in [(1, 1), (1, 16), (8, 64), (32, 128), (51, 99), (128, 256), (512, 512), (100000, 7)]:
        for resident in (256, 512):
            planes = nb.nb_march_planes(tiles, nz, resident, 64)
            assert 1 <= planes <= 64 and planes & (planes - 1) == 0
            cost = lambda p: -(-tiles * -(-nz // p) // resident) * (min(p, nz) + 0.75)  # noqa: E731
            assert cost(planes) == min(cost(2 ** k) for k in range(7))
    assert nb.nb_march_planes(8, 64, 512, 64) == 1      # 64^3: every compute unit has work
    assert nb.nb_march_planes(128, 256, 512, 64) == 64  # 256^3: one round of long marches
