"""Which candidate frames a ray walks, and in what order: what it counts
against the step limit, the frames a counted trace reports and the rays a
hit-buffer launch traces again, in launches that test the candidates one by
one and through the box hierarchy (needs the GPU)."""
import numpy as np
import pytest

import parity
from svogen import scenes

pytestmark = pytest.mark.gpu

CELL = 8.0      # edge of a part's cell: level 2 of a 32^3 world
LIMITED = -2    # the id of a ray that the step limit ended


def parts(n, places):
    """n parts, part s with its cell moved to places[s]: a slab over the
    cell's half at low z.  The world around them is one voxel."""
    cells = [(2, (s % 4, s // 4 % 4, s // 16)) for s in range(n)]
    occ = np.zeros((32, 32, 32), bool)
    for _, (x, y, z) in cells:
        occ[8 * x:8 * x + 8, 8 * y:8 * y + 8, 8 * z:8 * z + 4] = True
    occ[31, 31, 31] = True
    fwd = np.zeros((n, 3, 4), np.float32)
    fwd[:, [0, 1, 2], [0, 1, 2]] = 1.0
    fwd[:, :, 3] = np.asarray(places, np.float64) - CELL * np.array([c for _, c in cells])
    return scenes.from_occupancy(occ, cells, fwd.reshape(n, 12), name="parts")


def rays(origins, direction):
    d = np.asarray(direction, np.float64)
    r = np.zeros((len(origins), 8), np.float32)
    r[:, 0:3], r[:, 4:7], r[:, 7] = origins, d / np.linalg.norm(d), np.inf
    return r


@pytest.fixture(scope="module")
def ctx():
    import torch
    assert torch.cuda.is_available()
    from paper_1911_06001_amd import svo
    with svo.Context(0) as c:
        yield c


@pytest.fixture(params=[64, 1], ids=["one by one", "hierarchy"])
def limit(ctx, request):
    ctx.set_config(sorted_candidates=request.param)
    yield request.param
    ctx.set_config(sorted_candidates=0, step_limit=1 << 20)


def upload(ctx, sc):
    h = ctx.upload_scene(sc)
    ctx.set_transforms(h, sc.xform(0))
    st = ctx.scene_stats(h)
    assert st.n_candidates == sc.n_slots > 10    # (a table of up to 10 slots is always tested one by one)
    return h


def passed_by(n):
    """n parts in a row towards +y and +z, and rays across the row's x whose
    direction has no x: they miss the world, pass each cell's edge by up to
    0.4 and meet each cell's bounding sphere."""
    at = [(44.0, 40.0 + 10 * s, 40.0 + 10 * s) for s in range(n)]
    k = np.arange(64)
    return at, rays(np.stack([46.0 + k / 16.0, 28.1 + k / 200.0, np.full(64, 20.0)], 1), (0, 1, 1))


def test_parts_a_ray_passes_by_count_no_step(ctx, limit):
    """A selection that starts no walk is none: a ray that misses the world
    and every part needs one step, whatever its first tests met."""
    import torch
    at, r = passed_by(12)
    h = upload(ctx, parts(12, at))
    ctx.set_config(step_limit=1)
    out = ctx.trace(h, torch.from_numpy(r).cuda())
    torch.cuda.synchronize()
    assert bool((out.id == -1).all()), int((out.id == LIMITED).sum())
    ctx.free_scene(h)


def test_parts_a_ray_passes_by_keep_its_last_hit(ctx, limit):
    """The hit buffer traces a ray again only if a part may reach it; a
    direction along a coordinate plane widens no entry test but that plane's
    own."""
    import torch
    at, r = passed_by(12)
    sc = parts(12, at)
    h = upload(ctx, sc)
    dev = torch.from_numpy(r).cuda()
    out = ctx.trace(h, dev)
    ctx.set_transforms(h, sc.xform(0))
    again = torch.zeros(1, dtype=torch.int64, device="cuda")
    ctx.trace_reuse(h, dev, out, retraced=again)
    torch.cuda.synchronize()
    assert int(again) == 0
    assert bool((out.id == -1).all())
    ctx.free_scene(h)


def frames_walked(ctx, h, r):
    import torch
    out, counts, _ = ctx.trace_counted(h, torch.from_numpy(r).cuda())
    torch.cuda.synchronize()
    return out, counts[1].cpu().numpy()


@pytest.mark.parametrize("near,hidden", [(3, 9), (9, 3)])
def test_entries_that_differ_in_their_fifth_digit(ctx, limit, near, hidden):
    """Entries are compared in 32 bits: the part that is 0.06 nearer at a
    distance of 1,000 is walked first, and hides the other."""
    far = [(200.0 + 40 * s, 100.0, 900.0) for s in range(12)]   # (the hierarchy's leaves come in order of x)
    far[hidden] = (38.0, 40.0, 950.08)
    far[near] = (40.0, 40.0, 950.02)
    k = np.arange(64)
    r = rays(np.stack([41.0 + k / 16.0, 41.0 + k / 32.0, np.full(64, -50.0)], 1), (0, 0, 1))
    h = upload(ctx, parts(12, far))
    out, frames = frames_walked(ctx, h, r)
    assert bool((out.inst == near).all())
    assert (frames == 1).all(), frames
    ctx.free_scene(h)


@pytest.mark.parametrize("n", [11, 22, 60])      # over one, three and eight lists of seven
def test_the_nearest_of_a_row_is_walked_first(ctx, limit, n):
    """Rays against a row of n parts, whose list runs from the far end: each
    walks the nearest one and no other.  From the middle of the row too, where
    half of it lies behind."""
    h = upload(ctx, parts(n, [(50.0 + 10 * s, 40.0, 40.0) for s in range(n)]))
    k = np.arange(64)
    for x0, inst in ((100.0 + 10 * n, n - 1), (50.0 + 10 * (n // 2) - 1.0, n // 2 - 1)):
        o = np.stack([np.full(64, x0), 41.0 + k / 16.0, 41.0 + k / 32.0], 1)
        out, frames = frames_walked(ctx, h, rays(o, (-1, 0, 0)))
        assert bool((out.inst == inst).all())
        assert (frames == 1).all(), (x0, frames)
    ctx.free_scene(h)


@pytest.mark.parametrize("n", [11, 14, 15, 60])
def test_parts_entered_at_the_same_t_are_walked_once(ctx, limit, n):
    """Rays that start inside the empty halves of n overlapping parts and leave
    without a hit: every part is entered at tmin, and walked exactly once."""
    h = upload(ctx, parts(n, [(40.0 + 0.01 * s, 40.0, 40.0) for s in range(n)]))
    k = np.arange(64)
    o = np.stack([43.0 + k / 32.0, 43.0 + k / 64.0, np.full(64, 46.0)], 1)
    out, frames = frames_walked(ctx, h, rays(o, (0, 0.01, 1)))
    assert bool((out.id == -1).all())
    assert (frames == n).all(), frames
    ctx.free_scene(h)


def test_rays_from_anywhere_against_many_parts(ctx, oracle_lib):
    """Waves of unrelated rays, and of rays of several jobs, each finding its
    own way through the hierarchy over more than a hundred parts."""
    import torch
    from paper_1911_06001_amd import svo
    sc = scenes.tiny_scene(41, K=6, n_slots=120, nested=False, scale_range=(1.0, 3.0))
    assert sc.n_slots > 100
    r = scenes.random_rays(13, 3000, 0, 64)
    n = r.shape[0]
    h = upload(ctx, sc)
    dev = torch.from_numpy(r).cuda()
    new = lambda: svo.Hits(torch.full((n,), -7, dtype=torch.int32, device="cuda"),
                           torch.full((n,), -7, dtype=torch.int32, device="cuda"),
                           torch.full((n,), -7.0, device="cuda"), torch.full((n, 3), -7.0, device="cuda"))
    one, many = new(), new()
    ctx.trace_into(h, dev, one.id, one.t, one.inst, one.normal)
    cuts = [0, 1, 3, 20, 50, 51, 130, 700, 705, 1999, n]
    ctx.trace_batch([dict(scene=h, rays=dev[a:b], out_id=many.id[a:b], out_inst=many.inst[a:b], out_t=many.t[a:b],
                          out_normal=many.normal[a:b]) for a, b in zip(cuts, cuts[1:])])
    torch.cuda.synchronize()
    for k in ("id", "inst", "t", "normal"):
        assert torch.equal(getattr(one, k), getattr(many, k)), k
    ref = oracle_lib.trace_scene(sc, r, margin=True)
    st = parity.compare(parity.to_numpy(one), ref, ref.margin, r)
    parity.assert_parity(st)
    assert st["hits"] > 1000
    ctx.free_scene(h)


def test_a_batch_of_1998_frame_records_fits(ctx):
    """Two jobs of 999 frame records, eight of them candidates found through
    the hierarchy: tables that leave room for one wave's state."""
    import copy

    import torch
    from paper_1911_06001_amd import svo
    n, slots = 8, 998
    sc = copy.copy(parts(n, [(50.0 + 10 * s, 40.0, 40.0) for s in range(n)]))
    fwd = np.tile(np.eye(3, 4, dtype=np.float32).reshape(1, 12), (slots, 1))
    fwd[:n] = sc.xform(0)
    sc.slot_child = np.concatenate([sc.slot_child, np.zeros(slots - n, np.uint32)])
    sc.slot_cell = np.concatenate([sc.slot_cell, np.ones((slots - n, 4), np.float32)])
    k = np.arange(64)
    r = torch.from_numpy(rays(np.stack([np.full(64, 300.0), 41.0 + k / 16.0, 41.0 + k / 32.0], 1), (-1, 0, 0))).cuda()
    h = ctx.upload_scene(sc)
    ctx.set_transforms(h, fwd)
    assert ctx.scene_stats(h).n_candidates == n
    ctx.set_config(sorted_candidates=1)
    out = [svo.Hits(torch.full((64,), -7, dtype=torch.int32, device="cuda"),
                    torch.full((64,), -7, dtype=torch.int32, device="cuda"),
                    torch.full((64,), -7.0, device="cuda"), None) for _ in range(2)]
    ctx.trace_batch([dict(scene=h, rays=r, out_id=o.id, out_inst=o.inst, out_t=o.t) for o in out])
    torch.cuda.synchronize()
    ctx.set_config(sorted_candidates=0)
    for o in out:
        assert bool((o.inst == n - 1).all())
        assert bool((o.t == 300.0 - 50.0 - 10.0 * (n - 1) - CELL).all())
    ctx.free_scene(h)


@pytest.mark.parametrize("m", [1, 2, 6, 7, 8, 13, 14, 15])
def test_list_lengths_with_a_device_table(ctx, oracle_lib, limit, m):
    """m parts that overlap and twelve far away, so that the table is too large
    for the kernel arguments: rays that meet up to m of them, as a first trace
    and as a re-trace after the parts moved (lists hold seven)."""
    import torch
    from paper_1911_06001_amd import svo
    n = m + 12
    at = [(40.0 + 0.6 * s, 40.0 + 0.3 * (s % 5), 40.0 + 0.2 * (s % 3)) for s in range(m)]
    sc = parts(n, at + [(300.0 + 20 * s, 300.0, 300.0) for s in range(12)])
    moved = sc.xform(0).copy()
    moved.reshape(n, 3, 4)[:, :, 3] += 0.7
    r = scenes.random_rays(m, 2000, 38.0, 52.0)
    dev = torch.from_numpy(r).cuda()
    h = upload(ctx, sc)
    for fwd in (None, moved):
        out = svo.Hits(torch.full((2000,), -7, dtype=torch.int32, device="cuda"),
                       torch.full((2000,), -7, dtype=torch.int32, device="cuda"),
                       torch.full((2000,), -7.0, device="cuda"), torch.full((2000, 3), -7.0, device="cuda"))
        if fwd is None:
            ctx.trace_into(h, dev, out.id, out.t, out.inst, out.normal)
        else:
            ctx.trace_into(h, dev, out.id, out.t, out.inst, out.normal)
            ctx.set_transforms(h, fwd)
            ctx.trace_reuse(h, dev, out)
        torch.cuda.synchronize()
        ref = oracle_lib.trace_scene(sc, r, fwd=fwd, margin=True)
        st = parity.compare(parity.to_numpy(out), ref, ref.margin, r)
        parity.assert_parity(st)
        assert st["hits"] > 300
    ctx.free_scene(h)
