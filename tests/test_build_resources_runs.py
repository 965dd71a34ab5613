"""Per-lane scratch memory of the binned insert's and the run query's kernels,
as the compiler reports it with the library's own flags: their arrays are
indexed by constants and held in registers for every window length (6 to 32),
and an instantiation whose arrays went to scratch would run several times slower
with the same bits."""

import os
import shutil
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2606_24417_amd import build as B
from test_build_resources import _resources

SOURCES = ["kernels_binned.hip", "kernels_runs4.hip", "kernels_runs8.hip", "kernels_runs16.hip"]


@pytest.mark.skipif(shutil.which(B.hipcc()) is None and not os.path.exists(B.hipcc()), reason="no hipcc")
def test_run_kernels_use_no_scratch():
    with ThreadPoolExecutor(len(SOURCES)) as ex:
        found = dict(ex.map(_resources, SOURCES))
    for src, kernels in found.items():
        assert kernels, "no kernel resource report for %s" % src
        over = {k: v for k, v in kernels.items() if v > 0}
        assert not over, "%s: kernels using scratch memory: %s" % (src, over)
    # 39 front ends (w and class of m): two tiles of the bin kernel, and the run
    # query at H = 4 and at any H
    assert sum("bin_kernel" in k for k in found["kernels_binned.hip"]) == 2 * 39
    for src in SOURCES[1:]:
        assert sum("query_runs_kernel" in k for k in found[src]) >= 2 * 39
