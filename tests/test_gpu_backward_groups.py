"""The two-level adjoint with as many groups of rays as it takes in LDS, 16,384
ranges of 128 triangles and 16,384 instances, whose counters fill 128 KB in
one workgroup: gradients against the fixed-point atomic rows within two
float32 roundings, ray gradients bit for bit, and the same with only one of
the two outputs."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2603_00292_amd import workloads as wl

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -24
TRIANGLES, INSTANCES, RAYS = 1 << 21, 16384, 200003


def test_most_groups(monkeypatch):
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    rng = wl.rng_for(750)
    n = 1024   # n x n quads
    mv, mf = wl.grid_mesh(n, n, -1.0, 1.0, -1.0, 1.0, rng.normal(0.0, 0.002, (n + 1) ** 2))
    assert mf.shape[0] == TRIANGLES
    side = 128
    srt = np.zeros((INSTANCES, 10), np.float32)
    srt[:, 0:3] = rng.uniform(0.4, 0.6, (INSTANCES, 3))
    srt[:, 6] = 1.0
    srt[:, 7] = np.arange(INSTANCES) % side * 2.0
    srt[:, 9] = np.arange(INSTANCES) // side * 2.0
    o = np.stack([rng.uniform(-0.5, 2 * side - 1.5, RAYS), np.full(RAYS, 3.0),
                  rng.uniform(-0.5, 2 * side - 1.5, RAYS)], 1)
    d = np.tile([0.0, -1.0, 0.0], (RAYS, 1)) + rng.uniform(-0.05, 0.05, (RAYS, 3))
    rays = torch.from_numpy(wl.pack_rays(o, d)).cuda()
    g = torch.from_numpy(rng.standard_normal((RAYS, 3)).astype(np.float32)).cuda()
    V, I = torch.from_numpy(mv).cuda(), torch.from_numpy(mf.view(np.int32)).cuda()

    def run(ctx, vertices=True, frames=True):
        acc = api.Accel(ctx, [(V, I)], np.zeros(INSTANCES, np.uint32), srt, device_build=True)
        hits, inst = api.trace_closest(acc, rays, want_inst=True)
        dV = torch.zeros_like(V) if vertices else None
        dS = torch.zeros((INSTANCES, 10), device="cuda") if frames else None
        do, dd = api.trace_backward_instances(acc, rays, hits, inst, g, dV, dS)
        torch.cuda.synchronize()
        out = [None if t is None else t.cpu().numpy().astype(np.float64) for t in (dV, dS, do, dd)]
        ids = inst.cpu().numpy()
        acc.close()
        return out, ids

    ctx = api.Context(0)
    (dV, dS, do, dd), ids = run(ctx)
    hit = ids != -1
    print("hit fraction", hit.mean(), "instances hit", np.unique(ids[hit]).size, flush=True)
    assert hit.mean() > 0.1 and np.unique(ids[hit]).size > 8000
    for kw, k in (({"frames": False}, 0), ({"vertices": False}, 1)):
        one, _ = run(ctx, **kw)
        assert np.array_equal(one[k], (dV, dS)[k]) and np.array_equal(one[2], do) and np.array_equal(one[3], dd)
    monkeypatch.setenv("RT_BACKWARD_ATOMIC", "1")
    rows = api.Context(0)
    monkeypatch.delenv("RT_BACKWARD_ATOMIC")
    (bV, bS, bo, bd), _ = run(rows)
    assert np.array_equal(do, bo) and np.array_equal(dd, bd)
    for x, y, name in ((dV, bV, "vertices"), (dS, bS, "frames")):
        tol = 2 * EPS32 * np.maximum(np.abs(x), np.abs(y)) + 1e-9 * np.abs(x).max()
        print(name, "max err/tol", float((np.abs(x - y) / tol).max()), flush=True)
        assert (np.abs(x - y) <= tol).all()
    ctx.close()
    rows.close()
