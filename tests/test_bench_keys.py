"""Host logic of the benchmark's byte counts (no GPU): they follow the keys
that are emitted, which with PAPER boxes are fewer than the rectangles' tiles
that the plan reports, and every record binned by rows carries its spans."""
import types

import pytest
import torch  # noqa: F401  (before the library: the process must map one HIP runtime, torch's)

import bench
from paper_2505_05643_amd._lib import UG_FLAG_SCATTER


@pytest.mark.parametrize("box,flags,rows", [(0, 0, True), (0, 8, True), (0, UG_FLAG_SCATTER, False), (1, 0, False),
                                            (2, 0, True)])
def test_key_sizes(box, flags, rows):
    s = bench.key_sizes(types.SimpleNamespace(box_mode=box, flags=flags), 41)
    assert s == {"k": 41, "rows": rows}


def test_bytes_follow_the_emitted_keys():
    common = dict(n=10, p=4, r=100, t=16, m=1024, passes=1, w=1, g_sort=1, dslots=256)
    paper = types.SimpleNamespace(box_mode=0, flags=0)
    few, many = (dict(common, **bench.key_sizes(paper, k)) for k in (410, 690))
    for name, per_key in (("emit", 8), ("sort_hist", 4), ("sort_scatter", 16), ("record_adj", 32)):
        assert bench.kernel_bytes(name, **many) - bench.kernel_bytes(name, **few) == 280 * per_key
