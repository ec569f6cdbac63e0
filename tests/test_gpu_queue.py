"""The work queue around its edges: launches with fewer tiles than partitions
or waves (fixed claims only), a tile or a ray either side of one and two tiles
per wave, and claims larger than what a partition holds.  Every ray is written
exactly once and equals the oracle's."""
import numpy as np
import pytest

import parity
from svogen import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env(oracle_lib):
    import torch
    assert torch.cuda.is_available()
    from paper_1911_06001_amd import svo
    sc = scenes.noisy_sphere_d6()
    waves = torch.cuda.get_device_properties(0).multi_processor_count   # one wave per CU below
    rays = scenes.random_rays(9, 64 * (2 * waves + 65), 0, 64)
    ref = oracle_lib.trace_scene(sc, rays, margin=True)
    with svo.Context(0) as ctx:
        h = ctx.upload_scene(sc)
        ctx.set_transforms(h, sc.xform(0))
        yield torch, ctx, h, torch.from_numpy(rays).cuda(), ref, waves


def first(ref, n):
    class Cut:
        pass
    cut = Cut()
    for k in ("id", "inst", "t", "normal", "margin"):
        setattr(cut, k, getattr(ref, k)[:n])
    cut.margin_n = None if getattr(ref, "margin_n", None) is None else ref.margin_n[:n]
    return cut


@pytest.mark.parametrize("refill,claim", [(0, 1), (0, 2), (48, 2), (17, 64)])
@pytest.mark.parametrize("tiles,extra", [(0, 1), (1, 0), (1, 1), (64, -1), (64, 0), (64, 1), ("w", 0), ("w", 1),
                                         ("2w", -1), ("2w", 0), ("2w", 1), ("2w+64", 0)])
def test_every_ray_once(env, tiles, extra, refill, claim):
    torch, ctx, h, rays, ref, waves = env
    t = {"w": waves, "2w": 2 * waves, "2w+64": 2 * waves + 64}.get(tiles, tiles)
    n = 64 * t + extra
    ctx.set_config(waves_per_block=1, blocks_per_cu=1, refill_lanes=refill, claim_tiles=claim)
    part = rays[:n].contiguous()
    for _ in range(3):   # the same rays again: slow tiles first from the second launch on
        hits = ctx.trace(h, part)
    _, counts, _ = ctx.trace_counted(h, part)
    torch.cuda.synchronize()
    assert bool((counts[2] == 1).all())
    cut = first(ref, n)
    parity.assert_parity(parity.compare(parity.to_numpy(hits), cut, cut.margin))


@pytest.mark.parametrize("refill,claim", [(0, 1), (0, 2), (48, 2), (17, 64)])
@pytest.mark.parametrize("tiles,extra", [(0, 1), (1, 1), (64, 0), (64, 1), ("w", 0), ("w", 1), ("2w", -1), ("2w", 1),
                                         ("2w+64", 0)])
def test_every_launch_writes_every_ray(env, tiles, extra, refill, claim):
    """The product kernel into buffers filled before each of three launches of
    the same rays: the second has the slow-tile state, the third a list."""
    torch, ctx, h, rays, ref, waves = env
    from paper_1911_06001_amd import svo
    t = {"w": waves, "2w": 2 * waves, "2w+64": 2 * waves + 64}.get(tiles, tiles)
    n = 64 * t + extra
    ctx.set_config(waves_per_block=1, blocks_per_cu=1, refill_lanes=refill, claim_tiles=claim)
    part = rays[:n].contiguous()
    out = svo.Hits(torch.empty(n, dtype=torch.int32, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda"),
                   torch.empty(n, dtype=torch.float32, device="cuda"),
                   torch.empty((n, 3), dtype=torch.float32, device="cuda"))
    cut = first(ref, n)
    for launch in range(3):
        for x in (out.id, out.inst, out.t, out.normal):
            x.fill_(-77)
        ctx.trace_into(h, part, out.id, out.t, out.inst, out.normal)
        torch.cuda.synchronize()
        for x in (out.id, out.inst, out.t, out.normal):
            assert not bool((x == -77).any()), launch
        parity.assert_parity(parity.compare(parity.to_numpy(out), cut, cut.margin))
