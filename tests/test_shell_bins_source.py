"""The shell sums' LDS bins are cleared, added to and read by different lanes: the source orders every
such step explicitly (the race cannot be provoked: one wavefront's LDS operations keep their order)."""

import os
import re

from paper_2212_11024_amd import build as B


def _body(text, name):
    start = text.index("{", re.search(r"\b%s\(" % name, text).end())
    depth = 0
    for i in range(start, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[start:i]
    raise AssertionError(name)


def test_every_lds_step_of_the_bins_is_ordered():
    with open(os.path.join(B.CSRC, "flame_api.hip")) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    sync = _body(text, "void bins_sync")
    assert "__builtin_amdgcn_fence" in sync and "__builtin_amdgcn_wave_barrier" in sync
    for name in ("void bins_clear", "void bin_piece"):
        assert _body(text, name).rstrip().endswith("bins_sync();"), name
    for name in ("shell_bin_kernel", "transfer_bin_kernel"):
        body = _body(text, name)
        assert "bins_clear(" in body and not re.search(r"bins\[[^\]]*\]\s*=", body), name
