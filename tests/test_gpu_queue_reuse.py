"""Launches that share one scratch (queue heads, spill stack) one after another:
a batched plan launched on several streams without a wait between them, inside
a caller's graph and through its own graph, and accels of one context and of
two contexts through the process-wide array, all with more rays than the chip
takes at once.  Every launch answers as the same rays do in one ordinary
launch."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import to_gpu_scene
from paper_2603_00292_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 327,680 rays are 64 on each of 20 waves on 256 CUs: more go through the queues
N = 500003


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    ctx = api.Context(0)
    W = wl.random_triangles(n_tri=600, n_rays=N, k=730, half=0.05)
    acc = to_gpu_scene(api, torch, ctx, W.scene)
    rays = torch.from_numpy(W.rays).cuda()
    ref = api.trace_closest(acc, rays)[0].view(torch.int32).clone()
    torch.cuda.synchronize()
    yield torch, api, ctx, W, acc, rays, ref
    acc.close()
    ctx.close()


def test_plan_on_several_streams(gpu):
    torch, api, ctx, W, acc, rays, ref = gpu
    parts = [r.contiguous() for r in rays.split([350000, 1, N - 350001])]
    plan = api.BatchPlan(ctx, [acc] * 3, parts)
    streams = [torch.cuda.Stream() for _ in range(3)]
    for h in plan.hits:
        h.fill_(-1.0)
    torch.cuda.synchronize()
    for rep in range(9):
        with torch.cuda.stream(streams[rep % 3]):
            plan.launch()
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(plan.hits).view(torch.int32), ref)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        plan.launch()
    own = plan.graph_exec(streams[0])
    for go in (g.replay, lambda: api.graph_launch(own), plan.launch, g.replay, plan.launch):
        for h in plan.hits:
            h.fill_(-1.0)
        torch.cuda.synchronize()
        go()
        torch.cuda.synchronize()
        assert torch.equal(torch.cat(plan.hits).view(torch.int32), ref)
    plan.close()


def test_context_on_several_streams(gpu):
    """Launches of different grids on one context's scratch, queued without a
    wait between them."""
    torch, api, ctx, W, acc, rays, ref = gpu
    streams = [torch.cuda.Stream() for _ in range(3)]
    ns = [N, 65, 327681, N, 40001, N]
    outs = []
    parts = [rays[:n].contiguous() for n in ns]
    torch.cuda.synchronize()
    for k, n in enumerate(ns):
        with torch.cuda.stream(streams[k % 3]):
            outs.append(api.trace_closest(acc, parts[k])[0])
    torch.cuda.synchronize()
    for n, h in zip(ns, outs):
        assert torch.equal(h.view(torch.int32), ref[:n]), n


def test_captured_between_eager(gpu):
    """Closest and any hits captured into a caller's graph, replayed between
    launches on other streams: every replay and every launch is whole."""
    torch, api, ctx, W, acc, rays, ref = gpu
    occ = api.trace_any(acc, rays)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        hits, _ = api.trace_closest(acc, rays)
        any_hit = api.trace_any(acc, rays)
    streams = [torch.cuda.Stream() for _ in range(2)]
    for rep in range(5):
        hits.fill_(-1.0)
        any_hit.fill_(7)
        torch.cuda.synchronize()
        g.replay()
        if rep % 2:
            g.replay()
        torch.cuda.synchronize()
        assert torch.equal(hits.view(torch.int32), ref) and torch.equal(any_hit, occ), rep
        outs = []
        for s in streams[: 1 + rep % 2]:
            with torch.cuda.stream(s):
                outs.append(api.trace_closest(acc, rays)[0])
        torch.cuda.synchronize()
        for h in outs:
            assert torch.equal(h.view(torch.int32), ref), rep


def test_process_wide_scratch(gpu):
    """Contexts of different variants, so of different grids, one after another."""
    torch, api, ctx, W, acc, rays, ref = gpu
    for s, wg in ((8, 64), (16, 256), (32, 128), (16, 256)):
        c = api.Context(0, stack_entries=s, workgroup=wg)
        a = to_gpu_scene(api, torch, c, W.scene)
        for n in (N, 327681):
            h = torch.full((n, 4), -1.0, dtype=torch.float32, device="cuda")
            api.trace_closest_noalloc(a, rays[:n].contiguous(), h)
            torch.cuda.synchronize()
            assert torch.equal(h.view(torch.int32), ref[:n]), (s, wg, n)
        a.close()
        c.close()
