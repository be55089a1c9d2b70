"""Workgroups per launch: a grid dimension may not have 2^32 work-items, so
launches over more tiles than that go out in spans (no GPU needed)."""
import ctypes as C

import pytest

from paper_1010_4124_amd import lbm


@pytest.mark.parametrize("threads", [64, 256, 512, 768])
def test_span_is_the_largest_below_2_32_work_items(threads):
    L = lbm.lib()
    L.lbmi_launch_span.restype, L.lbmi_launch_span.argtypes = C.c_int64, [C.c_int]
    span = L.lbmi_launch_span(threads)
    assert span % 8 == 0 and span * threads < 1 << 32 <= (span + 8) * threads
    # a 1 x 33.6 M grid in tiles of 4 rows, 512 threads each, takes two launches
    if threads == 512:
        assert span < 33_600_000 // 4 <= 2 * span
