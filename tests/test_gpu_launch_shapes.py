"""How the traversal kernel gives out rays: up to 64 per resident wave in one
fixed share each, beyond that fixed shares and then chunks of eight queues of
tiles, whose counters the launch itself leaves at zero.  Ray counts at the
edges of these (one ray, around a wave, around the change to queues, a ragged
last tile) answer bit for bit as the same rays do in another launch, and the
largest launch lies in the oracle's sets on every ray; so do 64-bit node
addresses (used by accels whose nodes exceed 4 GiB; forced here), and the
other stack and workgroup variants."""
from __future__ import annotations

import os

import numpy as np
import pytest

from helpers import check_chunked, to_gpu_scene
from paper_2603_00292_amd import workloads as wl

pytestmark = pytest.mark.gpu

# 327,680 rays are 64 on each of 20 waves on 256 CUs
COUNTS = [700001, 1, 31, 64, 65, 1025, 32769, 327679, 327680, 327681, 400003]


def scene(two_level):
    if two_level:
        W = wl.aimed_instances(n_inst=8, n_rays=COUNTS[0], k=720)
        return W.scene, W.rays
    W = wl.random_triangles(n_tri=600, n_rays=COUNTS[0], k=721, half=0.05)
    return W.scene, W.rays


def run(api, torch, acc, rays, two_level):
    h, i = api.trace_closest(acc, rays, want_inst=two_level)
    o = api.trace_any(acc, rays)
    torch.cuda.synchronize()
    return h.view(torch.int32), o, i


@pytest.mark.parametrize("two_level", [False, True])
def test_ray_counts(orc, two_level):
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    ctx = api.Context(0)
    s, rays_h = scene(two_level)
    acc = to_gpu_scene(api, torch, ctx, s)
    rays = torch.from_numpy(rays_h).cuda()
    full = None
    for n in COUNTS + COUNTS[:1]:
        got = run(api, torch, acc, rays[:n].contiguous(), two_level)
        if full is None:
            full = got
        for a, b in zip(got, full):
            assert a is b is None or torch.equal(a, b[:n]), n
    S = orc.OracleScene.from_scene(s, accel=True)
    st = check_chunked(orc, S, rays_h, hits=full[0].cpu().numpy().view(np.float32), occ=full[1].cpu().numpy(),
                       inst=full[2].cpu().numpy().view(np.uint32) if two_level else None)
    print(st, flush=True)
    for stack, wg in ((8, 64), (32, 128), (8, 256)):
        ctx.set_variant(stack, wg)
        for n in (65, 400003):
            for a, b in zip(run(api, torch, acc, rays[:n].contiguous(), two_level), full):
                assert a is b is None or torch.equal(a, b[:n]), (stack, wg, n)
    acc.close()
    ctx.close()


@pytest.mark.parametrize("two_level", [False, True])
def test_batched_counts(two_level):
    """Batched plans, launched and replayed as a graph, at the same edges."""
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    ctx = api.Context(0)
    s, rays_h = scene(two_level)
    acc = to_gpu_scene(api, torch, ctx, s)
    rays = torch.from_numpy(rays_h).cuda()
    ref = api.trace_closest(acc, rays)[0].view(torch.int32)
    side = torch.cuda.Stream()
    for sizes in ((1, 5), (327675, 5), (327675, 6), (100000, 1, 299999, 63)):
        parts = [r.contiguous() for r in rays[: sum(sizes)].split(list(sizes))]
        plan = api.BatchPlan(ctx, [acc] * len(sizes), parts)
        g = plan.graph_exec(side)
        for go in (plan.launch, lambda: api.graph_launch(g), plan.launch, lambda: api.graph_launch(g)):
            for h in plan.hits:
                h.fill_(-1.0)
            go()
            torch.cuda.synchronize()
            assert torch.equal(torch.cat(plan.hits).view(torch.int32), ref[: sum(sizes)]), sizes
        plan.close()
    acc.close()
    ctx.close()


@pytest.mark.parametrize("two_level", [False, True])
@pytest.mark.parametrize("width", [2, 4, 8])
def test_wide_node_addresses(width, two_level):
    import torch

    from paper_2603_00292_amd import api

    torch.cuda.set_device(0)
    s, rays_h = scene(two_level)
    rays = torch.from_numpy(rays_h[:20000]).cuda()
    out = []
    for wide in ("0", "1"):
        os.environ["RT_WIDE_NODES"] = wide
        try:
            ctx = api.Context(0)
        finally:
            del os.environ["RT_WIDE_NODES"]
        acc = to_gpu_scene(api, torch, ctx, s, node_width=width)
        masks = torch.full((rays.shape[0],), 3, dtype=torch.int32, device="cuda")
        got = list(run(api, torch, acc, rays, two_level))
        got += api.trace_closest_ex(acc, rays, ray_masks=masks)[:1]
        got.append(api.trace_any_ex(acc, rays, ray_masks=masks))
        h, _, c = api.trace_all(acc, rays, 3, ray_masks=masks)
        got += [h, c]
        torch.cuda.synchronize()
        out.append(got)
        acc.close()
        ctx.close()
    for a, b in zip(*out):
        assert a is b is None or torch.equal(a.view(torch.uint8), b.view(torch.uint8))
