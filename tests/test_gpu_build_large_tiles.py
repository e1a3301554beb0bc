"""Device builds above 65,536 clusters, where a clustering pass takes its pairs
in tiles of 960 positions and changes to tiles of 192 further down the same
batch: a last tile of one position, exact duplicates (pairs chosen by hash
alone), every cluster a leaf of its own.  Checked as the smaller builds are:
bit for bit against a host build, with the counts of a whole tree."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2603_00292_amd import workloads as wl
from test_gpu_build_sizes import check, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [65537, 960 * 69 + 1, 200003])
def test_sizes(gpu, n):  # noqa: F811
    V, I = wl.random_triangle_soup(wl.rng_for(760 + n), n, 0.02)
    check(gpu, V, I)


@pytest.mark.parametrize("n", [70001])
def test_duplicates(gpu, n):  # noqa: F811
    V = np.tile(np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0.5]], np.float32), (n, 1))
    check(gpu, V, np.arange(3 * n, dtype=np.uint32).reshape(-1, 3), max_leaf_size=2)


def test_binary_nodes_of_one_triangle(gpu):  # noqa: F811
    V, I = wl.random_triangle_soup(wl.rng_for(761), 100003, 0.02)
    info = check(gpu, V, I, node_width=2, max_leaf_size=1)
    assert info["leaf_count"] == 100003 and info["node_count"] == 100002
