"""A wave of a closest-hit launch that finalizes its own hits remembers 64 ray
ranges and then leaves the rest to others.  With one workgroup on a CU, seven
of eight waves start on rays that cross 6,000 triangles each, and almost all
further rays are void: the other waves come to their limit while the slow ones
are still on their first share.  Every ray is answered as in launches of one
share a wave, bit for bit, on one level and on two."""
from __future__ import annotations

import os

import numpy as np
import pytest

from helpers import to_gpu_scene
from paper_2603_00292_amd import workloads as wl

pytestmark = pytest.mark.gpu

N = 1000003


def slow_scene(two_level):
    """6,000 parallel triangles that fill half of [0,1]^2, and one behind them
    over the other half; rays up the other half meet every box and only the
    last triangle."""
    n = 6000
    z = np.linspace(0.0, 1.0, n, dtype=np.float32)
    V = np.zeros((n + 1, 3, 3), np.float32)
    V[:n, 1, 0] = V[:n, 2, 1] = 1.0
    V[:n, :, 2] = z[:, None]
    V[n] = [[1, 0, 2], [1, 1, 2], [0, 1, 2]]
    mesh = wl.Mesh(V.reshape(-1, 3), np.arange(3 * (n + 1), dtype=np.uint32).reshape(-1, 3))
    if not two_level:
        return wl.Scene([mesh])
    srt = np.array([[1, 1, 1, 0, 0, 0, 1, 0, 0, 0], [1, 1, 1, 0, 0, 0, 1, 3, 0, 0]], np.float32)
    return wl.Scene([mesh], np.zeros(2, np.uint32), srt)


@pytest.mark.parametrize("two_level", [False, True])
def test_waves_at_their_range_limit(two_level):
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    waves = 4 * torch.cuda.get_device_properties(0).multi_processor_count
    rng = wl.rng_for(740)
    o = np.empty((N, 3))
    o[:, :2] = rng.uniform(0.8, 0.95, (N, 2))
    o[:, 2] = 1.5
    d = np.tile([0.0, 0.0, 1.0], (N, 1))
    i = np.arange(N)
    # 64 rays to a chunk and whole tiles to the first shares: those are the
    # first 64 * waves rays, a wave's in a row
    slow = (i < 64 * waves) & ((i >> 6) % 8 != 0)
    o[slow, 2] = -1.0
    d[~slow & (i % 640 != 0)] = 0.0   # void rays
    rays = torch.from_numpy(wl.pack_rays(o, d)).cuda()
    os.environ["RT_BLOCKS_PER_CU"] = "1"
    try:
        ctx = api.Context(0)
    finally:
        del os.environ["RT_BLOCKS_PER_CU"]
    acc = to_gpu_scene(api, torch, ctx, slow_scene(two_level))
    got = [api.trace_closest(acc, rays, want_inst=True) for _ in range(2)]
    ref = [api.trace_closest(acc, r.contiguous(), want_inst=True) for r in rays.split(64 * waves)]
    hits = torch.cat([h for h, _ in ref]).view(torch.int32)
    inst = torch.cat([j for _, j in ref])
    torch.cuda.synchronize()
    for h, j in got:
        assert torch.equal(h.view(torch.int32), hits) and torch.equal(j, inst)
    live = torch.from_numpy(d.any(1)).cuda()
    assert bool(((hits[:, 1] == 6000) == live).all()) and bool(((inst == 0) == live).all())
    acc.close()
    ctx.close()
