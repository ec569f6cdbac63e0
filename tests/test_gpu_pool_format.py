"""The device pool format: node words are re-encoded at upload (absolute child
starts; packed with the mask into one word up to 2^24 - 1 nodes, apart in
wider pools), so scenes on either side of that line, with far pointers, alone
and mixed in one batch, must match the oracle, which reads the upload
format."""
import copy

import numpy as np
import pytest

import parity
from svogen import scenes

pytestmark = pytest.mark.gpu

PACKED = 0xFFFFFF       # the largest pool whose words are packed
FAR = np.uint64(0xFFFFFF)


def stretched(sc, n_nodes):
    """sc with every node but the root moved to the end of a pool of n_nodes
    nodes (solid leaves in between), the root's children by far pointer."""
    shift = n_nodes - sc.nodes.shape[0]
    assert shift > 0 and sc.root == 0
    out = copy.copy(sc)
    nodes = np.full(n_nodes, np.uint64(0xFF112233) << np.uint64(32), np.uint64)
    root = int(sc.nodes[0])
    child = (root >> 8) & 0xFFFFFF
    nodes[0] = np.uint64(root & 0xFF) | (FAR << np.uint64(8)) | (np.uint64(child + shift) << np.uint64(32))
    nodes[1 + shift:] = sc.nodes[1:]
    out.nodes, out.slot_child = nodes, (sc.slot_child + np.uint32(shift)).astype(np.uint32)
    return out


def make(kind, n_nodes):
    # parts entered in place, or parts that are candidates
    sc = scenes.tiny_scene(17, K=5, n_slots=8, nested=True, scale_range=(0.3, 0.5) if kind == "inline" else (0.5, 2.0))
    return sc if n_nodes is None else stretched(sc, n_nodes)


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1911_06001_amd import svo
    with svo.Context(0) as c:
        yield c


@pytest.mark.parametrize("sorted_candidates", [0, 1])
@pytest.mark.parametrize("kind", ["inline", "candidates"])
@pytest.mark.parametrize("n_nodes", [None, PACKED, PACKED + 1])
def test_pool_sizes_around_the_packed_limit(ctx, oracle_lib, n_nodes, kind, sorted_candidates):
    import torch
    sc = make(kind, n_nodes)
    rays = scenes.random_rays(5, 3000, 0, 32)
    ctx.set_config(sorted_candidates=sorted_candidates)
    h = ctx.upload_scene(sc)
    ctx.set_transforms(h, sc.xform(0))
    got = parity.to_numpy(ctx.trace(h, torch.from_numpy(rays).cuda()))
    ctx.set_config(sorted_candidates=0)
    ref = oracle_lib.trace_scene(sc, rays, margin=True)
    st = parity.compare(got, ref, ref.margin, rays)
    parity.assert_parity(st)
    assert st["hits"] > 300
    # any node id may be shaded: its word 1 as it was uploaded
    ids = np.linspace(0, sc.nodes.shape[0], 64, dtype=np.uint32)
    ids[:8] = np.arange(8)
    ids[8:40] = sc.nodes.shape[0] - 1 - np.arange(32)
    img = ctx.shade(h, torch.from_numpy(ids.view(np.int32)).cuda(), 8, 8, tiled=False).cpu().numpy().view(np.uint32)
    word1 = (sc.nodes >> np.uint64(32)).astype(np.uint32)
    want = np.array([(word1[i] if i < sc.nodes.shape[0] else 0xFF402010) for i in ids], np.uint32)
    assert np.array_equal(img.ravel() & 0xFFFFFF, want & 0xFFFFFF)
    ctx.free_scene(h)


@pytest.mark.parametrize("sorted_candidates", [0, 1])
def test_packed_and_wide_pools_in_one_batch(ctx, oracle_lib, sorted_candidates):
    import torch
    from paper_1911_06001_amd import svo
    ctx.set_config(sorted_candidates=sorted_candidates)
    rays = scenes.random_rays(6, 1500, 0, 32)
    dev = torch.from_numpy(rays).cuda()
    runs = []
    for kind, n in (("inline", None), ("candidates", PACKED + 1), ("candidates", PACKED), ("inline", PACKED + 1)):
        sc = make(kind, n)
        h = ctx.upload_scene(sc)
        k = rays.shape[0]
        out = svo.Hits(torch.empty(k, dtype=torch.int32, device="cuda"), torch.empty(k, dtype=torch.int32, device="cuda"),
                       torch.empty(k, dtype=torch.float32, device="cuda"), torch.empty((k, 3), dtype=torch.float32, device="cuda"))
        runs.append((sc, h, out))
    jobs = [dict(scene=h, fwd=sc.xform(0), rays=dev, out_id=o.id, out_inst=o.inst, out_t=o.t, out_normal=o.normal)
            for sc, h, o in runs]
    with ctx.plan([h for _, h, _ in runs], max_jobs=4, max_frames=64) as plan:
        for launch in ("batch", "plan"):
            for _, _, o in runs:
                o.id.zero_()
            if launch == "batch":
                ctx.trace_batch(jobs)
            else:
                plan.set_jobs(jobs)
                plan.launch()
            torch.cuda.synchronize()
            for sc, _, o in runs:
                ref = oracle_lib.trace_scene(sc, rays, margin=True)
                parity.assert_parity(parity.compare(parity.to_numpy(o), ref, ref.margin, rays))
    ctx.set_config(sorted_candidates=0)
    for _, h, _ in runs:
        ctx.free_scene(h)


@pytest.mark.parametrize("path", ["one by one", "hierarchy"])
@pytest.mark.parametrize("kind", ["inline", "candidates"])
@pytest.mark.parametrize("n_nodes", [None, PACKED, PACKED + 1])
def test_pool_sizes_with_a_device_table(ctx, oracle_lib, n_nodes, kind, path):
    """One-job launches of 12 parts, whose table is too large for the kernel
    arguments, on either candidate path of either word format."""
    import torch
    from paper_1911_06001_amd import svo
    sc = scenes.tiny_scene(17, K=5, n_slots=12, nested=True, scale_range=(0.3, 0.5) if kind == "inline" else (0.8, 2.0))
    assert sc.n_slots == 12
    if n_nodes is not None:
        sc = stretched(sc, n_nodes)
    rays = scenes.random_rays(8, 3000, 0, 32)
    n = rays.shape[0]
    dev = torch.from_numpy(rays).cuda()
    h = ctx.upload_scene(sc)
    ctx.set_transforms(h, sc.xform(0))
    st = ctx.scene_stats(h)
    assert st.n_inline > 2 if kind == "inline" else st.n_candidates > 8
    ctx.set_config(sorted_candidates=64 if path == "one by one" else 1)
    out = svo.Hits(torch.full((n,), -7, dtype=torch.int32, device="cuda"),
                   torch.full((n,), -7, dtype=torch.int32, device="cuda"),
                   torch.full((n,), -7.0, device="cuda"), torch.full((n, 3), -7.0, device="cuda"))
    ctx.trace_into(h, dev, out.id, out.t, out.inst, out.normal)
    again, _, _ = ctx.trace_counted(h, dev)
    torch.cuda.synchronize()
    ctx.set_config(sorted_candidates=0)
    for k in ("id", "inst", "t", "normal"):
        assert torch.equal(getattr(out, k), getattr(again, k)), k
    ref = oracle_lib.trace_scene(sc, rays, margin=True)
    stats = parity.compare(parity.to_numpy(out), ref, ref.margin, rays)
    parity.assert_parity(stats)
    assert stats["hits"] > 300
    ctx.free_scene(h)


def test_pool_without_a_root_shades_as_uploaded(ctx):
    """A pool without a root is not checked; any of its words may be shaded."""
    import torch
    nodes = np.random.default_rng(3).integers(0, 1 << 63, 4096, dtype=np.uint64) * np.uint64(2) + np.uint64(1)
    h = ctx.upload(nodes, 0xFFFFFFFF, (0, 0, 0), 1.0, 20, np.zeros(0, np.uint32), np.zeros((0, 4), np.float32))
    ids = torch.arange(4096, dtype=torch.int32, device="cuda")
    img = ctx.shade(h, ids, 64, 64, tiled=False).cpu().numpy().view(np.uint32).ravel()
    want = (nodes >> np.uint64(32)).astype(np.uint32)
    assert np.array_equal(img & 0xFFFFFF, want & 0xFFFFFF)
    ctx.free_scene(h)
