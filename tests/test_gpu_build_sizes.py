"""Device builds at the sizes where the clustering changes its kernels: one
workgroup up to 1,024 clusters, tiles of 1,024 above, batches of eight passes,
lists of exact duplicates (pairs chosen by hash alone), and collapses deeper
than one batch of levels.  Answers do not depend on the tree, so a device
build answers bit for bit like a host build; node and leaf counts are those
of a whole tree."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import to_gpu_scene
from paper_2603_00292_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    yield torch, api, api.Context(0)
    torch.cuda.synchronize()


def check(gpu, V, I, **build):
    torch, api, ctx = gpu
    rays = torch.from_numpy(wl.box_rays(wl.rng_for(360), 4099, -0.5, 1.5)).cuda()
    outs = []
    for dev in (False, True):
        acc = to_gpu_scene(api, torch, ctx, wl.Scene([wl.Mesh(V, I)]), device_build=dev, **build)
        hits, _ = api.trace_closest(acc, rays)
        outs.append((hits.cpu().numpy().view(np.uint32), api.trace_any(acc, rays).cpu().numpy(), acc.info))
        acc.close()
    (hh, oh, _), (hd, od, info) = outs
    assert np.array_equal(hh, hd) and np.array_equal(oh, od)
    assert info["triangle_count"] == I.shape[0]
    leaf = build.get("max_leaf_size", 4)
    assert info["leaf_count"] * leaf >= I.shape[0]
    # a tree with that many leaves, no node with more than `width` children
    assert (info["node_count"] - 1) + info["leaf_count"] <= info["node_count"] * build.get("node_width", 4)
    return info


@pytest.mark.parametrize("n", [1, 2, 3, 64, 65, 513, 1023, 1024, 1025, 2047, 2049, 40001])
def test_sizes(gpu, n):
    V, I = wl.random_triangle_soup(wl.rng_for(361 + n), n, 0.1)
    check(gpu, V, I)


@pytest.mark.parametrize("n", [2, 1024, 1025, 9001])
def test_duplicates(gpu, n):
    V = np.tile(np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0.5]], np.float32), (n, 1))
    check(gpu, V, np.arange(3 * n, dtype=np.uint32).reshape(-1, 3), max_leaf_size=2)


def test_binary_nodes_of_one_triangle(gpu):
    """40,001 triangles in binary nodes with one triangle a leaf: every
    merge is a node, and the tree is deeper than sixteen levels."""
    V, I = wl.random_triangle_soup(wl.rng_for(362), 40001, 0.02)
    info = check(gpu, V, I, node_width=2, max_leaf_size=1)
    assert info["max_depth"] > 16 and info["leaf_count"] == 40001 and info["node_count"] == 40000
