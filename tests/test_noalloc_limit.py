"""The sizes that include/akf.h gives for the no-allocation step's array: each
fits with the default scan block or, where the header says so, with blocks of 4."""
import ctypes as C
import os
import re

import pytest

from paper_2303_00301_amd import _lib
from tests.test_capi_host import _fake_model

HEADER = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "akf.h")


def test_sizes_named_by_the_header():
    lib = _lib.load()
    text = re.sub(r"\s*\n \*\s*", " ", open(HEADER).read())
    (rule,) = re.findall(r"With block = 0 the scan block is .*?\.\s+64 MiB covers, e\.g\., (.*?)\. ", text)
    sizes = [tuple(map(int, p)) for p in re.findall(r"dx = (\d+) at N = (\d+)", rule)]
    assert len(sizes) == 3
    by_default = 0
    for d, N in sizes:
        need = [lib.akf_mh_workspace_bytes(C.byref(_fake_model(N=N, dx=d, dy=d)), 2, b) for b in (0, 4)]
        assert 0 < min(need) <= _lib.NOALLOC_SCRATCH_BYTES, (d, N, need)
        by_default += need[0] <= _lib.NOALLOC_SCRATCH_BYTES
    assert 0 < by_default < len(sizes)  # both branches of the rule are among them


@pytest.mark.parametrize("block", [0, 4])
def test_a_problem_past_the_limit_is_past_it_either_way(block):
    m = _fake_model(N=4096, dx=64, dy=32)
    assert _lib.load().akf_mh_workspace_bytes(C.byref(m), 2, block) > _lib.NOALLOC_SCRATCH_BYTES
