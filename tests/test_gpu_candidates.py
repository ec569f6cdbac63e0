"""The candidate frames of a ray are listed after its walk of the world, at
most eight at a time, by a sphere test of each or by one walk of the box
hierarchy: with parts that nearly all overlap, rays meet one, eight, nine and
up to forty of them, as a first trace, as a re-trace after the parts moved and
as jobs of a batch; against the oracle (needs the GPU)."""
import numpy as np
import pytest

import parity
from svogen import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1911_06001_amd import svo
    with svo.Context(0) as c:
        yield c


@pytest.mark.parametrize("limit", [1, 64])      # from two parts on the hierarchy, always one by one
@pytest.mark.parametrize("n_slots", [1, 2, 3, 8, 9, 40])
def test_list_lengths(ctx, oracle_lib, n_slots, limit):
    import torch
    from paper_1911_06001_amd import svo
    sc = scenes.tiny_scene(23, K=5, n_slots=n_slots, nested=False, scale_range=(4.0, 6.0))
    there, here = sc.xform(0), sc.xform(0).copy()
    there.reshape(-1, 3, 4)[:, :, 3] += 1.5
    rays = scenes.random_rays(n_slots, 2000, 0, 32)
    n = rays.shape[0]
    dev = torch.from_numpy(rays).cuda()
    ctx.set_config(sorted_candidates=limit)
    h = ctx.upload_scene(sc)
    new = lambda: svo.Hits(*(torch.empty(s, dtype=t, device="cuda") for s, t in (
        (n, torch.int32), (n, torch.int32), (n, torch.float32), ((n, 3), torch.float32))))
    got = {}
    ctx.set_transforms(h, there)
    out = new()
    ctx.trace_into(h, dev, out.id, out.t, out.inst, out.normal)
    ctx.set_transforms(h, here)
    got["re-trace"] = ctx.trace_reuse(h, dev, out)
    got["trace"] = ctx.trace(h, dev)
    jobs = [dict(scene=h, fwd=f, rays=dev, out_id=o.id, out_inst=o.inst, out_t=o.t, out_normal=o.normal)
            for f, o in ((there, new()), (here, got.setdefault("batch", new())))]
    ctx.trace_batch(jobs)
    torch.cuda.synchronize()
    ctx.set_config(sorted_candidates=0)
    ref = oracle_lib.trace_scene(sc, rays, margin=True)
    for how, o in got.items():
        print("[gpu-candidates]", n_slots, limit, how, flush=True)
        st = parity.compare(parity.to_numpy(o), ref, ref.margin, rays)
        parity.assert_parity(st)
        assert st["hits"] > 300
    assert len(np.unique(ref.inst)) >= min(n_slots, 8)
    ctx.free_scene(h)
