"""Workspaces and plans of the spectral diagnostics at scratch limits, on the host with the device's memory
and the transform library replaced by counters."""

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2212_11024_amd import _lib as L

HERE = os.path.dirname(os.path.abspath(__file__))
GIB = 1 << 30


@pytest.fixture(scope="module")
def ss(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("ss") / "ss.so")
    subprocess.run([hipcc, "-O1", "-std=c++17", "-fPIC", "-shared", "--offload-host-only", "-fuse-cuid=none", "-x", "hip",
                    os.path.join(HERE, "hostcheck", "spectral_setup.hip"), "-o", out, "-L/opt/rocm/lib", "-lhipfft",
                    "-Wl,-rpath,/opt/rocm/lib", "-Wl,-Bsymbolic"], check=True, stderr=subprocess.DEVNULL)
    lib = ctypes.CDLL(out)
    lib.ss_new.restype = ctypes.c_void_p
    lib.ss_new.argtypes = [ctypes.c_int] * 3 + [ctypes.c_size_t, ctypes.c_double]
    lib.ss_room.argtypes = [ctypes.c_size_t]
    lib.ss_setup.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t]
    lib.ss_batch.argtypes = [ctypes.c_void_p]
    lib.ss_held.restype = ctypes.c_size_t
    return lib


NX, NY, NZ, SHELLS = 97, 65, 50, 4
HALF = 16 * (NX // 2 + 1) * NY * NZ                      # bytes of one half spectrum
FIELDS = 6 * HALF + 9 * 8 * NX * NY * NZ                 # the energy transfer's own arrays
SUMS = 8 * SHELLS * (3250 + 1)                           # partial sums of one term: a block per row of 49 entries


def _ok(ss, c, batch):
    assert ss.ss_batch(c) == batch and ss.ss_bad_releases() == 0


def test_enough_memory_takes_three_components(ss):
    c = ss.ss_new(NX, NY, NZ, GIB, 4.0)
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_OK
    _ok(ss, c, 3)
    before = ss.ss_held()
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_OK and ss.ss_held() == before


@pytest.mark.parametrize("transfer", [0, FIELDS])
def test_one_component_uses_all_that_three_held(ss, transfer):
    """Just enough for one component, its plans' work areas and the call's other arrays: the memory that the
    attempt with three took is given back."""
    need = HALF + 4 * HALF * (2 if transfer else 1) + SUMS * (4 if transfer else 1) + transfer
    c = ss.ss_new(NX, NY, NZ, need, 4.0)
    assert ss.ss_setup(c, SHELLS, transfer) == L.FLAME_OK
    _ok(ss, c, 1)
    assert ss.ss_held() <= need


def test_a_spectrum_before_does_not_take_the_transfers_memory(ss):
    need = HALF + 8 * HALF + 5 * SUMS + FIELDS
    c = ss.ss_new(NX, NY, NZ, need + HALF, 4.0)          # room for a spectrum of three, not for both
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_OK
    assert ss.ss_setup(c, SHELLS, FIELDS) == L.FLAME_OK
    _ok(ss, c, 1)


def test_no_memory_is_reported_and_a_later_call_tries_again(ss):
    c = ss.ss_new(NX, NY, NZ, HALF // 2, 0.0)
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_E_NOMEM
    assert ss.ss_setup(c, SHELLS, FIELDS) == L.FLAME_E_NOMEM
    ss.ss_room(GIB)
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_OK
    assert ss.ss_setup(c, SHELLS, FIELDS) == L.FLAME_OK
    assert ss.ss_bad_releases() == 0


@pytest.mark.parametrize("failures", [1, 2])
def test_a_plan_without_the_stream_is_not_used(ss, failures):
    """The stream cannot be set for the plans of three components, and then not for those of one: the call
    fails, nothing is kept of the plan, and the next call makes it anew."""
    c = ss.ss_new(NX, NY, NZ, GIB, 0.0)
    ss.ss_fail_streams(failures)
    assert ss.ss_setup(c, SHELLS, 0) == (L.FLAME_OK if failures == 1 else L.FLAME_E_HIP)
    assert ss.ss_plans() == (1 if failures == 1 else 0)
    assert ss.ss_setup(c, SHELLS, 0) == L.FLAME_OK
    assert ss.ss_plans() == 1
    _ok(ss, c, 1)


@pytest.mark.parametrize("n,work_factor,batch", [(256, 0.0, 3), (512, 0.0, 3), (512, 1.0, 1), (420, 1.0, 3), (300, 4.0, 3),
                                                 (331, 4.0, 1), (576, 0.0, 1)])
def test_three_components_are_kept_up_to_4_gib_with_their_work_area(ss, n, work_factor, batch):
    c = ss.ss_new(n, n, n, 64 * GIB, work_factor)
    half = 16 * (n // 2 + 1) * n * n
    for transfer in (0, 6 * half + 72 * n ** 3):
        assert ss.ss_setup(c, SHELLS, transfer) == L.FLAME_OK
        _ok(ss, c, batch)
        spectra = batch * half * (1 + work_factor)       # one work area for both plans
        assert batch == 1 or spectra <= 4 * GIB
        assert abs(ss.ss_held() - spectra - transfer) < 8 << 20
