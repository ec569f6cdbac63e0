"""Compositing at the sizes where its quotients and tile edges can go wrong:
images of partial tiles only, the most samples and AO rays, and ids beyond
the pool; whole numbers, so equal to the oracle bit for bit (needs the GPU)."""
import numpy as np
import pytest

import oracle
from svogen import camera as cam
from svogen import scenes as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,samples,tiled,k,ambient", [
    (1, 1, 1, True, 1, 0), (7, 5, 3, True, 64, 333), (8, 8, 1, True, 0, 200), (9, 17, 7, True, 3, 1),
    (1, 65, 2, False, 5, 999), (333, 3, 1, True, 7, 1000), (5, 3, 1024, True, 64, 500), (5, 3, 1024, False, 63, 123)])
def test_shade_at_edges(W, H, samples, tiled, k, ambient):
    import torch
    assert torch.cuda.is_available()
    from paper_1911_06001_amd import svo
    sc = S.fbm_terrain_d10()
    leaves = np.nonzero((sc.nodes & 0xFFFFFFFF) == 0)[0]
    rng = np.random.default_rng(W * 1000 + H)
    n = W * H * samples
    ids = rng.choice(leaves, n).astype(np.uint32)
    miss = rng.random(n) < 0.3
    ids[miss] = rng.choice(np.array([0xFFFFFFFF, sc.nodes.size], np.uint32), int(miss.sum()))
    ao = np.where(rng.random(n * k) < 0.5, np.uint32(0xFFFFFFFF), np.uint32(3)).astype(np.uint32) if k else None
    ctx = svo.Context(0)
    h = ctx.upload_scene(sc)
    dev = lambda x: None if x is None else torch.from_numpy(x.view(np.int32)).cuda()
    img = ctx.shade(h, dev(ids), W, H, samples=samples, tiled=tiled, ao_id=dev(ao), k=k, ambient_permille=ambient,
                    background=0xFF603010)
    got = img.cpu().numpy().view(np.uint32)
    ctx.close()
    pix = cam.pixel_order(W, H, "tiles" if tiled else "rows")
    ref = oracle.shade(sc.nodes, ids, ao, W, H, samples, k, ambient, 0xFF603010, pix)
    assert np.array_equal(got.reshape(ref.shape), ref)
