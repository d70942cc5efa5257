"""Private memory of the marching kernels of the curl-stencil route, read on the host from the kernel metadata
of a gfx950 compile: a node's populations stay in registers (a workgroup of 512 threads caps them at 256)."""

import os
import shutil

import pytest

from paper_2212_11024_amd import build as B
from test_kernel_resources import _kernel_metadata

needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"),
                                 reason="hipcc is not installed")


@needs_hipcc
@pytest.mark.parametrize("src,kernel,count,bound", [("flame_step.hip", "step_zmarch", 45, 20),
                                                    ("flame_api.hip", "stencil_march_kernel", 18, 0)])
def test_marching_kernels_keep_the_node_in_registers(src, kernel, count, bound, tmp_path):
    meta = {k: v for k, v in _kernel_metadata(src, tmp_path).items() if kernel in k}
    assert len(meta) == count, len(meta)
    for k, (private, vgpr) in meta.items():
        # FP64: a few spilled registers in the odd in-place step, nothing more
        assert private <= (bound if "Id" in k else 0) and vgpr <= 512, (k, private, vgpr)
