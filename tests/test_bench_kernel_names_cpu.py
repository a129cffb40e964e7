"""What the benchmark says of a row follows what ran: the share of steps in pairs, and the library's own constants."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


@pytest.mark.parametrize("n,pairs,sc1,name", [(1024, 0.98, False, "k_sweep<float, false>"), (128, 0.8, False, "k_pair_tiles<float>"),
                                              (1024, 0.0, False, "k_step<float, 8, 2, 0, false, false>"), (2048, 1.0, False, "k_sweep<float, true>"),
                                              (1024, 1.0, True, "k_sweep_sc1<float, false>")])
def test_kernel_names(n, pairs, sc1, name):
    assert bench.kernel_name("f32", 8, 1, 2, np.zeros((n, n), np.uint8), pairs, sc1) == name


def test_bytes_per_launch_follow_the_share_of_pairs():
    r = [bench.roofline("k", "none.md", 1000, 1000, "f32", 1.0, pairs) for pairs in (0.0, 1.0, 0.5)]
    assert [x["steps_per_launch"] for x in r] == [1.0, 2.0, 1.333]
    assert r[1]["achieved"] == pytest.approx(r[0]["achieved"] / 2, abs=0.1)


def test_constants_come_from_the_kernel_sources():
    m = np.ones((28, 28), np.uint8)
    m[0, 0] = m[27, 27] = 0
    assert bench.library_constant("SMALL_MAX_TILES") == 768 and bench.pair_tiles(m) == 2
