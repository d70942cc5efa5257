"""The rules by which launches are shaped, on the host, at the sizes where both sides were timed."""

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2212_11024_amd import _lib as L

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def lr(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("lr") / "lr.so")
    subprocess.run([hipcc, "-O2", "-std=c++17", "-fPIC", "-shared", "--offload-host-only", "-x", "hip",
                    os.path.join(HERE, "hostcheck", "launch_rules.hip"), "-o", out], check=True, stderr=subprocess.DEVNULL)
    return ctypes.CDLL(out)


def test_unforced_fp32_stencil_steps_run_one_workgroup_per_compute_unit(lr):
    assert [lr.lr_one_group_per_cu(s, f) for s in (L.FLAME_F32, L.FLAME_F64, L.FLAME_F16) for f in (0, 1)] == \
        [1, 0, 0, 0, 0, 0]


@pytest.mark.parametrize("value,plain,hinted", [
    (4, [(64,) * 3, (112,) * 3, (118,) * 3, (130,) * 3, (132,) * 3, (160,) * 3, (200,) * 3, (512,) * 3],
     [(120,) * 3, (122,) * 3, (128,) * 3, (161, 130, 99), (64, 64, 512), (512, 64, 64)]),
    (8, [(48,) * 3, (88,) * 3, (94,) * 3, (112,) * 3, (128,) * 3, (512,) * 3], [(96,) * 3, (98,) * 3, (100,) * 3, (104,) * 3]),
    (2, [(128,) * 3, (152,) * 3, (160,) * 3, (256,) * 3], [])])
def test_in_place_stores_take_the_side_that_was_faster(lr, value, plain, hinted):
    assert [lr.lr_nt_stores(0, 0, value, *g) for g in plain] == [0] * len(plain)
    assert [lr.lr_nt_stores(0, 0, value, *g) for g in hinted] == [1] * len(hinted)


@pytest.mark.parametrize("two,value,hinted,reserved", [
    # sizes, whether the lattice's stores take the hint, whether LDS is reserved
    (0, 4, {64: 0, 96: 0, 112: 0, 116: 0, 124: 1, 128: 1, 132: 0, 160: 0, 256: 0, 512: 0},
     {64: 0, 96: 0, 112: 0, 116: 1, 128: 0, 132: 1, 144: 1, 160: 1, 224: 1, 256: 1, 512: 1}),
    (0, 8, {64: 0, 88: 0, 96: 1, 108: 1, 112: 1, 116: 1, 124: 0, 128: 0, 200: 0, 256: 0}, {64: 0, 128: 0, 256: 0}),
    (0, 2, {96: 0, 128: 0, 160: 0, 256: 0}, {96: 0, 128: 0, 144: 1, 160: 1, 256: 1, 384: 1}),
    (1, 4, {64: 1, 128: 1, 256: 1}, {64: 0, 104: 0, 112: 0, 136: 1, 160: 1, 256: 1, 512: 1}),
    (1, 2, {128: 1, 256: 1}, {128: 0, 144: 1, 160: 1, 256: 1}),
    (1, 8, {96: 1}, {96: 0, 256: 0})])
def test_state_saving_steps_take_the_side_that_was_faster(lr, two, value, hinted, reserved):
    assert {n: lr.lr_nt_stores(two, 1, value, n, n, n) for n in hinted} == hinted
    assert {n: int(lr.lr_reserved_lds(two, 1, value, n, n, n) > 0) for n in reserved} == reserved


def test_plain_steps_reserve_lds_from_2_to_the_25_fp32_nodes(lr):
    for two in (0, 1):
        got = {n: lr.lr_reserved_lds(two, 0, 4, n, n, n) for n in (256, 320, 336, 512)}
        assert got == {256: 0, 320: 0, 336: 50000, 512: 50000}
        assert lr.lr_reserved_lds(two, 0, 8, 512, 512, 512) == 0 and lr.lr_reserved_lds(two, 0, 2, 512, 512, 512) == 0
